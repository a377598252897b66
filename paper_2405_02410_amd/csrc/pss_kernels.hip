// HIP kernels of the pseudo-spectral stochastic step for gfx950.
//
// One 2D step (eq:timeupdate and the six-step list after it) is two kernels:
//
//   update kernel (lines along y, one or more packed columns per block)
//     forward y-FFT of every product channel  -> N_hat(kx, ky)       (step 4)
//     Philox4x32-10 + Box-Muller noise per mode, in registers        (step 5)
//     phi <- (phi + dt sum M N_hat + sigma xi) / (1 - dt L)          (step 6)
//     de-alias mask, inverse y-FFT of every factor field  -> V       (steps 2-3)
//   x kernel (lines along x, RB rows per block, two real rows per complex FFT)
//     inverse x-FFT of V (C2R) -> u(x, y); products sum c prod u^p   (step 3)
//     forward x-FFT (R2C) -> channel arrays for the next step        (step 4)
//
// The spectral arrays use the packed half-spectrum layout described in
// pss_plan.h: column 0 holds X(kx=0) + i X(kx=Nx/2).  Line transforms are the
// register/LDS transforms of pss_fft.h: a forward transform takes its input in
// digit-reversed order and returns natural order (dit), an inverse transform
// takes natural order and returns digit-reversed order (dif), so every
// per-mode computation sees natural mode order.  A line is held by
// consecutive threads.
//
// Position order.  The arrays that pass between the kernels of a step (the
// de-aliased factors V and the product channels N, and their adjoint
// counterparts) hold, along the update axis, position p = t + m*T the value
// of the digit-reversed index D(t) + m*T.  The update kernel then reads and
// writes them contiguously, and the x kernel (and the 3D y pass), whose work
// does not depend on the coordinate along that axis, simply treat positions
// as rows.  The state and the arrays of the transform modes (uploads,
// downloads) stay in natural order; those gather or scatter at D(t) + m*T.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pss_device.h"
#include "pss_fft.h"
#include "pss_kernels.h"
#include "pss_plan.h"

namespace pss {

// ----------------------------------------------------------------- twiddles
// Copy of the twiddle table into LDS, in two halves so that the caller can
// issue its own loads in between: every thread loads its (at most P) entries
// at once, then stores them.  The blocks hold at least L/P threads, so P
// entries per thread cover the table.  The caller puts a block barrier
// between the store and the first transform.
template <int L, int P>
__device__ __forceinline__ void load_twiddles(float2 (&w)[P], const float2* __restrict__ src, int tid, int nthr) {
    // unconditional loads (the index wraps, L is a power of two) keep the
    // memory counter exact for the loads the caller issues next
#pragma unroll
    for (int k = 0; k < P; ++k) w[k] = src[(tid + k * nthr) & (L - 1)];
}
template <int L, int P>
__device__ __forceinline__ const float2* store_twiddles(float2* dst, const float2 (&w)[P], int tid, int nthr) {
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = tid + k * nthr;
        if (i < L) dst[i] = w[k];
    }
    return dst;
}

// The twiddles of a kernel's line transforms: load() issues the reads next to
// the kernel's first data loads, ready() ends before the first transform (a
// block barrier only where the table is staged in LDS), get() goes to
// dif / dit.
template <class FFT, int L, int P, int FORM = fft_tw_form(L, P)>
struct Twiddles;
template <class FFT, int L, int P>
struct Twiddles<FFT, L, P, kTwRegs> {
    typename FFT::Regs r;
    __device__ __forceinline__ void load(const float2* __restrict__ tw_g, int t, int, int) { r.load(tw_g, t); }
    __device__ __forceinline__ void ready(float2*, int, int) {}
    __device__ __forceinline__ const typename FFT::Regs& get() const { return r; }
};
template <class FFT, int L, int P>
struct Twiddles<FFT, L, P, kTwSplit> {
    static constexpr int N1 = fft_tw_elems(L, P), PER = (N1 + FFT::T - 1) / FFT::T;
    static_assert(N1 == L / FFT::Split::R0, "the table is that of the second stage");
    typename FFT::Split r;
    float2 e[PER];
    __device__ __forceinline__ void load(const float2* __restrict__ tw_g, int t, int tid, int nthr) {
        r.load(tw_g, t);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            e[k] = gload_at(tw_g, static_cast<uint32_t>(((tid + k * nthr) & (N1 - 1)) * FFT::Split::R0));
    }
    __device__ __forceinline__ void ready(float2* lds, int tid, int nthr) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (tid + k * nthr < N1) lds[tid + k * nthr] = e[k];
        r.p = lds;
        __syncthreads();
    }
    __device__ __forceinline__ const typename FFT::Split& get() const { return r; }
};
template <class FFT, int L, int P>
struct Twiddles<FFT, L, P, kTwTable> {
    float2 w[P];
    typename FFT::Table tab;
    __device__ __forceinline__ void load(const float2* __restrict__ tw_g, int, int tid, int nthr) {
        load_twiddles<L, P>(w, tw_g, tid, nthr);
    }
    __device__ __forceinline__ void ready(float2* lds, int tid, int nthr) {
        tab.p = store_twiddles<L, P>(lds, w, tid, nthr);
        __syncthreads();
    }
    __device__ __forceinline__ const typename FFT::Table& get() const { return tab; }
};

// Sum of NV per-thread FP64 values over the block in a fixed order (a
// shuffle tree inside each wave, then the waves in index order), added by
// thread 0 into this block's own slot[0..NV).  Launches with the same grid
// add into the same slots in stream order, so the slots, and a fixed-order
// sum over them, do not depend on how the blocks are scheduled.  Every thread
// of the block calls it; the block is whole waves or a part of one.  old: the
// slot's values, which thread 0 read at the kernel's start (read here, they
// would be a memory latency at its very end).
template <int NV>
__device__ __forceinline__ void block_sum_to_slot(double (&v)[NV], const double (&old)[NV],
                                                  double* __restrict__ slot) {
    __shared__ double red[64 * NV];
    const int nt = blockDim.x, tid = threadIdx.x;
    const bool waves = (nt & 63) == 0;
    if (waves) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v[i] += __shfl_xor(v[i], o, 64);
        if ((tid & 63) == 0)
#pragma unroll
            for (int i = 0; i < NV; ++i) red[(tid >> 6) * NV + i] = v[i];
    } else {
#pragma unroll
        for (int i = 0; i < NV; ++i) red[tid * NV + i] = v[i];
    }
    __syncthreads();
    if (tid == 0) {
        const int n = waves ? nt >> 6 : nt;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            double acc = 0.0;
            for (int w = 0; w < n; ++w) acc += red[w * NV + i];
            slot[i] = old[i] + acc;
        }
    }
}

// ---------------------------------------------------------- exchange layout
// Where the arrays that pass between the column kernels and the x kernel
// (products N, factors V, the transform modes' in / out, the adjoint's
// counterparts) hold packed column c at row y of a 2D lattice.  Tiles of
// several columns (tc > 1): as the state, [ctile][y][TC].  One-column tiles:
// groups of four rows, [y/4][c][4].  A column is then 32-byte pieces and a
// row pair half of such pieces side by side: a kernel of either direction
// uses at least a quarter (columns) or half (rows) of the cache lines that it
// fetches, where whole columns, [c][y], gave the x kernel 16 bytes of each
// 128-byte line (1024^2: the gather took 1.4 us of the x launch).
// Offsets are 32-bit in 2D (a packed plane has at most 2^23 elements), so
// that they add to a scalar base in the load itself.
template <class I>
struct Exch {
    I c0;       // element of (c, y = 0)
    I ystride;  // from y to y + 1 (groups: from y to y + 4)
    bool grp;   // groups of four rows
    __device__ __forceinline__ I at(int y) const {
        return grp ? c0 + static_cast<I>(y >> 2) * ystride + static_cast<I>(y & 3) : c0 + static_cast<I>(y) * ystride;
    }
    // from y to y + n, n a multiple of four where rows are grouped
    __device__ __forceinline__ I step(int n) const { return static_cast<I>(grp ? n >> 2 : n) * ystride; }
};
// column c = ct * tc + cc of a 2D lattice of L rows
__device__ __forceinline__ Exch<uint32_t> exch_column(const Geo& geo, int ct, int cc, int L) {
    Exch<uint32_t> e;
    e.grp = geo.grp != 0;
    e.c0 = static_cast<uint32_t>(geo.grp ? ct * 4 : ct * L * geo.tc + cc);
    e.ystride = static_cast<uint32_t>(geo.grp ? geo.ntile * 4 : geo.tc);
    return e;
}

// ----------------------------------------------------------------- modes
struct ModeQ {
    float q2;
    float invq;  // 1/|q| (0 at q = 0)
    float iq[3];
};

// signed index of mode i on an axis of even length n (Nyquist read as -n/2)
__device__ __forceinline__ int signed_mode(int i, int n) { return i < (n >> 1) ? i : i - n; }

__device__ __forceinline__ ModeQ mode_q(int nx, int ny, int nz, const float (&qs)[3], int kx, int ky, int kz) {
    ModeQ m;
    const float qx = static_cast<float>(kx) * qs[0];
    const float qy = static_cast<float>(ky) * qs[1];
    const float qz = static_cast<float>(kz) * qs[2];
    m.q2 = qx * qx + qy * qy + qz * qz;
    m.iq[0] = (kx == -(nx >> 1)) ? 0.f : qx;
    m.iq[1] = (ky == -(ny >> 1)) ? 0.f : qy;
    m.iq[2] = (nz > 1 && kz == -(nz >> 1)) ? 0.f : qz;
    m.invq = m.q2 > 0.f ? 1.f / sqrtf(m.q2) : 0.f;
    return m;
}
__device__ __forceinline__ ModeQ mode_q(const DevPlan& p, int kx, int ky, int kz) {
    return mode_q(p.n[0], p.n[1], p.n[2], p.qs, kx, ky, kz);
}

// monomials with 1/|q| or i q_i factors, evaluated only by the kernel
// variants built for plans that have them
__device__ __forceinline__ float2 eval_general(const DevOp& op, const ModeQ& q) {
    const float q2 = q.q2, invq = q.invq, iqx = q.iq[0], iqy = q.iq[1], iqz = q.iq[2];
    float re = 0.f, im = 0.f;
    for (int i = 0; i < op.n; ++i) {
        const DevMono mo = op.m[i];
        float s = mo.coef;
        for (int e = 0; e < mo.q2; ++e) s *= q2;
        for (int e = 0; e < mo.invq; ++e) s *= invq;
        for (int e = 0; e < mo.ix; ++e) s *= iqx;
        for (int e = 0; e < mo.iy; ++e) s *= iqy;
        for (int e = 0; e < mo.iz; ++e) s *= iqz;
        switch (mo.ipow) {
            case 0: re += s; break;
            case 1: im += s; break;
            case 2: re -= s; break;
            default: im -= s; break;
        }
    }
    return make_float2(re, im);
}

// The pure q^2 part of an operator, read as one block.  Reading coefficient
// by coefficient behind a test of the degree makes every coefficient a scalar
// load of its own that the next one waits for, each about a microsecond on a
// cold cache: a step's operators were some thirty such waits in a row.
struct OpPoly {
    float c[PSS_MAXPOW + 1];
    int deg;
};
__device__ __forceinline__ OpPoly op_poly(const DevOp& op) {
    OpPoly r;
#pragma unroll
    for (int j = 0; j <= PSS_MAXPOW; ++j) r.c[j] = op.poly[j];
    r.deg = op.deg;
    return r;
}
// keep a uniform value in scalar registers from here on (the compiler would
// move its load down to the use, behind a barrier)
__device__ __forceinline__ void hold(int& x) {
    x = __builtin_amdgcn_readfirstlane(x);
    asm volatile("" : "+s"(x));
}
__device__ __forceinline__ void hold(uint32_t& x) {
    int v = static_cast<int>(x);
    hold(v);
    x = static_cast<uint32_t>(v);
}
__device__ __forceinline__ void hold(float& x) {
    int v = __float_as_int(x);
    hold(v);
    x = __int_as_float(v);
}
__device__ __forceinline__ void hold(OpPoly& o) {
#pragma unroll
    for (int j = 0; j <= 4; ++j) hold(o.c[j]);
    hold(o.deg);
}

// what is computed from x after this is computed here, not ahead of a loop or
// a transform (where its registers would be held)
template <class I>
__device__ __forceinline__ void fresh(I& x) {
    asm volatile("" : "+v"(x));
}

// sum_j c[j] (q^2)^j for P modes.  The coefficients above the degree are
// zeros, so starting at a fixed power gives c[deg] exactly when it is reached
// and the value does not depend on which of the three lengths is taken.
template <int N, int P>
__device__ __forceinline__ void horner_n(const OpPoly& op, const float (&q2)[P], float (&out)[P]) {
#pragma unroll
    for (int m = 0; m < P; ++m) out[m] = op.c[N];
#pragma unroll
    for (int j = N - 1; j >= 0; --j) {
#pragma unroll
        for (int m = 0; m < P; ++m) out[m] = fmaf(out[m], q2[m], op.c[j]);
    }
}
template <int P>
__device__ __forceinline__ void horner_p(const OpPoly& op, const float (&q2)[P], float (&out)[P]) {
    if (op.deg <= 2) {
        horner_n<2>(op, q2, out);
    } else if (op.deg <= 4) {
        horner_n<4>(op, q2, out);
    } else {
        horner_n<PSS_MAXPOW>(op, q2, out);
    }
}
template <int P>
__device__ __forceinline__ void horner_p(const DevOp& op, const float (&q2)[P], float (&out)[P]) {
    horner_p(op_poly(op), q2, out);
}
__device__ __forceinline__ float horner(const OpPoly& op, float q2) {
    const float q[1] = {q2};
    float r[1];
    horner_p(op, q, r);
    return r[0];
}
__device__ __forceinline__ float horner(const DevOp& op, float q2) { return horner(op_poly(op), q2); }

// sum_m coef (q^2)^a |q|^-b (i qx)^cx (i qy)^cy (i qz)^cz: Horner over the
// pure q^2 part, then the listed general monomials (GEN: the plan has some;
// without them the kernel is built without the out-of-line call, which would
// split the unrolled mode loops into separately scheduled pieces)
template <bool GEN>
__device__ __forceinline__ float2 eval_op(const DevOp& op, const ModeQ& q) {
    const float re = horner(op, q.q2);
    if constexpr (GEN) {
        if (op.n != 0) {
            const float2 g = eval_general(op, q);
            return make_float2(re + g.x, g.y);
        }
    }
    return make_float2(re, 0.f);
}

// the same for P modes at once: the monomial list is walked once, so its
// loads and uniform branches are paid per line and not per mode
template <int P>
__device__ __forceinline__ void eval_op_p(const DevOp& op, const float (&q2)[P], const ModeQ (&q)[P],
                                          float2 (&out)[P]) {
    float re[P];
    horner_p(op, q2, re);
#pragma unroll
    for (int m = 0; m < P; ++m) out[m] = make_float2(re[m], 0.f);
    if (op.n == 0) return;
    float gr[P], gi[P];
#pragma unroll
    for (int m = 0; m < P; ++m) gr[m] = gi[m] = 0.f;
    for (int i = 0; i < op.n; ++i) {
        const DevMono mo = op.m[i];
        float s[P];
#pragma unroll
        for (int m = 0; m < P; ++m) s[m] = mo.coef;
        for (int e = 0; e < mo.q2; ++e) {
#pragma unroll
            for (int m = 0; m < P; ++m) s[m] *= q[m].q2;
        }
        for (int e = 0; e < mo.invq; ++e) {
#pragma unroll
            for (int m = 0; m < P; ++m) s[m] *= q[m].invq;
        }
        for (int e = 0; e < mo.ix; ++e) {
#pragma unroll
            for (int m = 0; m < P; ++m) s[m] *= q[m].iq[0];
        }
        for (int e = 0; e < mo.iy; ++e) {
#pragma unroll
            for (int m = 0; m < P; ++m) s[m] *= q[m].iq[1];
        }
        for (int e = 0; e < mo.iz; ++e) {
#pragma unroll
            for (int m = 0; m < P; ++m) s[m] *= q[m].iq[2];
        }
        if (mo.ipow & 1) {
#pragma unroll
            for (int m = 0; m < P; ++m) gi[m] = mo.ipow == 1 ? gi[m] + s[m] : gi[m] - s[m];
        } else {
#pragma unroll
            for (int m = 0; m < P; ++m) gr[m] = mo.ipow == 0 ? gr[m] + s[m] : gr[m] - s[m];
        }
    }
#pragma unroll
    for (int m = 0; m < P; ++m) out[m] = make_float2(re[m] + gr[m], gi[m]);
}

// 1 / (1 - dt L(q)), complex (operators with odd i q_i powers)
__device__ __forceinline__ float2 cinv_implicit(float dt, float2 L) {
    const float ar = 1.f - dt * L.x, ai = -dt * L.y;
    const float d = 1.f / (ar * ar + ai * ai);
    return make_float2(ar * d, -ai * d);
}

__device__ __forceinline__ bool mask_keep(const DevMask& mk, int kx, int ky, int kz) {
    if (mk.shape == 2) return true;
    if (mk.shape == 1) {
        bool k = true;
        if (mk.h[0]) k = k && (mk.den * abs(kx) < mk.num * mk.h[0]);
        if (mk.h[1]) k = k && (mk.den * abs(ky) < mk.num * mk.h[1]);
        if (mk.h[2]) k = k && (mk.den * abs(kz) < mk.num * mk.h[2]);
        return k;
    }
    const int64_t s = mk.w[0] * kx * kx + mk.w[1] * ky * ky + mk.w[2] * kz * kz;
    return s * mk.den2 < mk.rhs;
}

// What the noise of one field takes from the plan
struct NoiseKey {
    uint32_t k0, k1, step;
    int fid;
    float amp_pair, amp_self;
};
__device__ __forceinline__ NoiseKey noise_key(const DevPlan& p, int f, uint32_t step) {
    return NoiseKey{p.key0, p.key1, step, p.fid[f], p.amp_pair, p.amp_self};
}
// Scaled unit white noise sigma(q) xi_hat(k) of field f at step `step` for a
// mode with full-spectrum linear index lin and negative-mode index lneg, and
// noise strength D(q) (Sec. "Adding noise").  PAIR: the mode is known not to
// be its own negative.
template <bool PAIR = false>
__device__ __forceinline__ float2 noise_value(const NoiseKey& n, uint32_t lin, uint32_t lneg, float D) {
    const uint32_t c = lin < lneg ? lin : lneg;
    const uint4 w = philox4x32_10(make_uint4(c, n.step, static_cast<uint32_t>(n.fid), 0u), n.k0, n.k1);
    const float2 g = box_muller(w.x, w.y);
    const float sd = __builtin_amdgcn_sqrtf(fmaxf(D, 0.f));
    if constexpr (!PAIR) {
        if (lin == lneg) return make_float2(n.amp_self * sd * g.x, 0.f);
    }
    const float a = n.amp_pair * sd;
    return lin == c ? make_float2(a * g.x, a * g.y) : make_float2(a * g.x, -a * g.y);
}
__device__ __forceinline__ float2 noise_value(const DevPlan& p, int f, uint32_t step, uint32_t lin, uint32_t lneg,
                                              float D) {
    return noise_value(noise_key(p, f, step), lin, lneg, D);
}
template <bool GEN>
__device__ __forceinline__ float2 noise_mode(const DevPlan& p, int f, uint32_t step, uint32_t lin, uint32_t lneg,
                                             const ModeQ& q) {
    return noise_value(p, f, step, lin, lneg, eval_op<GEN>(p.noise_op[f], q).x);
}

// full-spectrum linear index and its negative for signed mode indices
__device__ __forceinline__ void mode_lin(int nx, int ny, int nz, int kx, int ky, int kz, uint32_t& lin,
                                         uint32_t& lneg) {
    auto at = [&](int x, int y, int z) { return (static_cast<uint32_t>(z) * ny + y) * nx + x; };
    const int ux = kx & (nx - 1), uy = ky & (ny - 1), uz = kz & (nz - 1);
    lin = at(ux, uy, uz);
    lneg = at((nx - ux) & (nx - 1), (ny - uy) & (ny - 1), (nz - uz) & (nz - 1));
}

// f(integral_constant<int, I>) for I = 0 .. N-1, unrolled at compile time
template <int I, int N, class F>
__device__ __forceinline__ void static_for_from(F& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for_from<I + 1, N>(f);
    }
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_from<0, N>(f);
}

// Element f of a register array, f a runtime (block-uniform) field index.
// Written with bit masks rather than a chain of conditional copies: the
// compiler folds such a chain back into an indexed access, which moves the
// whole array to scratch memory.
template <int NF, int P>
__device__ __forceinline__ float2 pick(const float2 (&a)[NF][P], int f, int m) {
    if constexpr (NF == 1) return a[0][m];
    uint32_t rx = 0u, ry = 0u;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const uint32_t mk = f == i ? 0xffffffffu : 0u;
        rx |= __float_as_uint(a[i][m].x) & mk;
        ry |= __float_as_uint(a[i][m].y) & mk;
    }
    return make_float2(__uint_as_float(rx), __uint_as_float(ry));
}

// a[f][m] += v, f a runtime field index: every element takes v or +0 (bit
// masks, for the reason given at pick)
template <int NF, int P>
__device__ __forceinline__ void add_to(float2 (&a)[NF][P], int f, int m, float2 v) {
    if constexpr (NF == 1) {
        if (f == 0) a[0][m] = cadd(a[0][m], v);
        return;
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const uint32_t mk = f == i ? 0xffffffffu : 0u;
        a[i][m].x += __uint_as_float(__float_as_uint(v.x) & mk);
        a[i][m].y += __uint_as_float(__float_as_uint(v.y) & mk);
    }
}

// ------------------------------------------------------------ update kernel
// Lines along the last axis u (y in 2D, z in 3D).  A block holds TC packed
// columns x TO values of the other index o (y in 3D; none in 2D); the T
// threads of line (cc, lo) are consecutive, thread t keeps slot u = t + m*T
// of the line in v[m].  The state and the channel inputs are
// [o][ctile][u][TC]; the factor outputs V go to [ctile][u][TC] in 2D and to
// [u][ctile][o][TC] (the y-pass layout) in 3D.
//
// Which modes a line holds (signed indices):
//   c >= 1           : (c, u, -) in 2D, (c, o, u) in 3D
//   c = 0, 0<o<Ny/2  : (0, o, u)                          (3D)
//   c = 0, o>Ny/2    : (-Nx/2, Ny-o, u)                   (3D)
//   packed line (c = 0 in 2D; c = 0, o in {0, Ny/2} in 3D), slot form:
//     slot u in (0, L/2)  : kx = 0 at u
//     slot u in (L/2, L)  : kx = -Nx/2 at L - u
//     slots 0 and L/2     : (Re of kx = 0, Re of kx = -Nx/2), both real
// Transforms of a packed line see S(u) = phi(0,u) + i phi(Nx/2,u); the slot
// form is converted to and from it through one LDS line (block-uniform
// barriers; a block holds at most one packed line, its first).
// LDS: TC*TO line-transform regions | one exchange line of L | twiddles of L
// (P = 16 only; up to 8 points a thread keep them in registers).
//
// What bounds a 2D launch of one lattice is latency: 1024^2 is two blocks per
// CU and one round, so the launch lasts as long as one block's chain.  Cycle
// stamps along that chain (2.4 GHz): 1000 for the kernel arguments, 1700 to
// 5000 for the plan's scalars and the first loads, 2400 for the noise, 1300
// for each transform, 2000 for operators, update and mask.  Hence: every read
// is issued at the top (the plan as blocks of scalar loads held in registers,
// 35 waits in a row before), the de-aliasing limits come from a table (two
// 64-bit divisions a line before), and the self-conjugate modes of column 0
// are evaluated in four lanes (one thread's serial tail before, on the block
// that the launch waits for).  64^2: 8.0 -> 5.5 us, 1024^2: 10.2 -> 8.4 us a
// launch; with general operators (walked once per line instead of once per
// mode) KPZ 22.8 -> 12.5 us and Model H 69 -> 30 us.
//
// Long lines (2048, 4096) run in many rounds and are bound by how many waves
// hide the memory: see EARLY below and fft_one_buffer.  4096^2: 135 -> 85 us
// (2.9 TB/s), the x kernel 93 -> 53.5 us; a cap of 128 registers for four
// waves per SIMD spills (86.3 us), as it does in 3D (144 -> 273 us).

// packed line: S(u), S(L-u) -> slot value of u (the forward direction)
template <int L>
__device__ __forceinline__ float2 to_slot(int u, float2 a, float2 b) {
    if (u == 0 || u == (L >> 1)) return a;
    return u < (L >> 1) ? make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y))   // phi(0, u)
                        : make_float2(0.5f * (a.y + b.y), 0.5f * (a.x - b.x));  // phi(Nx/2, L-u)
}

// packed line: slot values of u and L-u -> S(u) = phi(0,u) + i phi(Nx/2,u)
template <int L>
__device__ __forceinline__ float2 from_slot(int u, float2 s1, float2 s2) {
    if (u == 0 || u == (L >> 1)) return s1;
    return u < (L >> 1) ? make_float2(s1.x - s2.y, s1.y + s2.x)   // phi0(u) + i phiN(u)
                        : make_float2(s2.x + s1.y, s1.x - s2.y);  // conj phi0(L-u) + i conj phiN(L-u)
}

// The modes of one line, decided once per thread: for slot u the signed
// index along the line is w(u), the fixed indices are those of the line
// (plain) or of the slot's half (packed: kx = 0 below L/2, -Nx/2 above).
struct LineModes {
    bool packed;
    int kx, ky;        // fixed indices of a plain line (3D: ky; 2D: ky unused)
    float qq;          // q_x^2 (+ q_y^2 in 3D) of a plain line
    float qqN;         // packed line: the same with kx = -Nx/2 (kx = 0 gives qq0)
    float qq0;
    float qs;          // q scale of the line axis
    uint32_t lstride;  // linear-index stride of the line axis
    uint32_t yx, yxn;  // linear-index parts of the fixed indices and of their negatives
    uint32_t yx0, yxN; // packed line: the same for kx = 0 and kx = -Nx/2 (negation keeps them)

};

// slot u (not a pair slot) of a line -> w, q^2, lin, lneg.  The line's
// description is taken by value so that it stays in registers.
template <int L>
__device__ __forceinline__ void slot_at(const LineModes lm, int u, float& q2, uint32_t& lin, uint32_t& lneg) {
    const bool upper = lm.packed && u > (L >> 1);
    const int w = lm.packed ? (upper ? L - u : u) : (u < (L >> 1) ? u : u - L);
    const float ql = static_cast<float>(w) * lm.qs;
    q2 = fmaf(ql, ql, lm.packed ? (upper ? lm.qqN : lm.qq0) : lm.qq);
    const uint32_t uw = static_cast<uint32_t>(w) & (L - 1), un = static_cast<uint32_t>(-w) & (L - 1);
    lin = uw * lm.lstride + (lm.packed ? (upper ? lm.yxN : lm.yx0) : lm.yx);
    lneg = un * lm.lstride + (lm.packed ? (upper ? lm.yxN : lm.yx0) : lm.yxn);
}

template <int L, int DIM>
__device__ __forceinline__ LineModes line_modes(int nx, int ny, const float (&qs)[3], bool packed, int kx_l,
                                                int ky_l) {
    LineModes lm;
    lm.packed = packed;
    lm.kx = kx_l;
    lm.ky = ky_l;
    const float qx = static_cast<float>(kx_l) * qs[0];
    const float qy = DIM == 3 ? static_cast<float>(ky_l) * qs[1] : 0.f;
    const float qxN = static_cast<float>(nx >> 1) * qs[0];
    lm.qq = fmaf(qx, qx, qy * qy);
    lm.qq0 = qy * qy;
    lm.qqN = fmaf(qxN, qxN, qy * qy);
    lm.qs = qs[DIM == 2 ? 1 : 2];
    lm.lstride = DIM == 2 ? static_cast<uint32_t>(nx) : static_cast<uint32_t>(nx) * ny;
    const uint32_t ux = static_cast<uint32_t>(kx_l) & (nx - 1), uxn = static_cast<uint32_t>(-kx_l) & (nx - 1);
    const uint32_t uy = DIM == 3 ? (static_cast<uint32_t>(ky_l) & (ny - 1)) : 0u;
    const uint32_t uyn = DIM == 3 ? (static_cast<uint32_t>(-ky_l) & (ny - 1)) : 0u;
    lm.yx = uy * nx + ux;
    lm.yxn = uyn * nx + uxn;
    // packed lines: kx = 0 or Nx/2 are their own negatives (mod Nx); in 3D
    // the packed lines have ky = 0 or -Ny/2, also their own negatives
    lm.yx0 = uy * nx;
    lm.yxN = uy * nx + (nx >> 1);
    return lm;
}

// the two real self-conjugate modes (kx = 0 and kx = -Nx/2) of slot u in
// {0, L/2} of a packed line: signed index w of the line axis
template <int DIM>
__device__ __forceinline__ void pair_modes(int ky_l, int u, int L, int& ky, int& kz) {
    const int w = u == 0 ? 0 : -(L >> 1);
    if (DIM == 2) {
        ky = w;
        kz = 0;
    } else {
        ky = ky_l;
        kz = w;
    }
}

// The four self-conjugate modes of a packed line (kx in {0, -Nx/2}, w in
// {0, -L/2}), which its slots 0 and L/2 hold in pairs.  Their operators and
// noise are evaluated side by side, mode j = lane & 3, and the thread that
// holds the two slots (the block's first) takes the four results from lanes 0
// to 3: evaluated in turn by that thread alone they were the longest chain of
// the launch, on the one block that every other waits for.
struct Self {
    ModeQ q;             // of the mode of this lane
    uint32_t lin, lneg;
};
struct Four {
    float v[4];
};
__device__ __forceinline__ Four four_lanes(float x) {
    Four r;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        r.v[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));
    return r;
}
template <int L, int DIM>
__device__ __forceinline__ Self self_modes(int nx, int ny, int nz, const float (&qs)[3], int ky_pack, int tid) {
    Self s;
    int ky, kz;
    pair_modes<DIM>(ky_pack, (tid & 2) ? (L >> 1) : 0, L, ky, kz);
    const int kx = (tid & 1) ? -(nx >> 1) : 0;
    s.q = mode_q(nx, ny, nz, qs, kx, ky, kz);
    mode_lin(nx, ny, nz, kx, ky, kz, s.lin, s.lneg);
    return s;
}
// v (pair slots m = 0 and P/2) times the real parts c of an operator there
template <int P>
__device__ __forceinline__ void pair_scale(const Four& c, const float2 (&v)[P], float2& lo, float2& hi) {
    static_assert(P >= 2, "slots 0 and L/2 lie in one thread");
    lo = make_float2(c.v[0] * v[0].x, c.v[1] * v[0].y);
    hi = make_float2(c.v[2] * v[P / 2].x, c.v[3] * v[P / 2].y);
}

// What the lines of a block have in common, for the per-mode operators
template <int P, bool LANES>
struct LineCtx {
    float q2[P];      // of the slots (pair slots: unused)
    bool first_wave;  // the wave holding the block's packed line, if it has one
    bool pair_lane;   // the thread holding that line's slots 0 and L/2
    Self self[LANES ? 1 : 4];  // first wave only: this lane's mode, or all four
};
// f at the four self-conjugate modes (first wave only): one per lane, or, on
// lines held by fewer than four threads, all of them in every thread
template <int P, bool LANES, class F>
__device__ __forceinline__ Four self_eval(const LineCtx<P, LANES>& cx, F&& f) {
    if constexpr (LANES) {
        return four_lanes(f(cx.self[0]));
    } else {
        Four r;
#pragma unroll
        for (int j = 0; j < 4; ++j) r.v[j] = f(cx.self[j]);
        return r;
    }
}

// mode q of slot u of a line, for the general-monomial operators
template <int L, int DIM>
__device__ __forceinline__ ModeQ slot_q(int nx, int ny, int nz, const float (&qs)[3], const LineModes lm, int u) {
    const bool upper = lm.packed && u > (L >> 1);
    const int w = lm.packed ? (upper ? L - u : u) : (u < (L >> 1) ? u : u - L);
    const int kx = lm.packed ? (upper ? -(nx >> 1) : 0) : lm.kx;
    return DIM == 2 ? mode_q(nx, ny, nz, qs, kx, w, 0) : mode_q(nx, ny, nz, qs, kx, lm.ky, w);
}

// acc[target] += op v on the slots of a line
template <bool GEN, int NF, int P, bool LANES>
__device__ __forceinline__ void accumulate(float2 (&acc)[NF][P], int target, const float2 (&v)[P], const DevOp& op,
                                           const OpPoly& poly, const LineCtx<P, LANES>& cx,
                                           const ModeQ (&qv)[GEN ? P : 1]) {
    float2 d[P];
    if constexpr (GEN) {
        float2 M[P];
        eval_op_p(op, cx.q2, qv, M);
#pragma unroll
        for (int m = 0; m < P; ++m) d[m] = cmul(M[m], v[m]);
    } else {
        float M[P];
        horner_p(poly, cx.q2, M);
#pragma unroll
        for (int m = 0; m < P; ++m) d[m] = cscale(v[m], M[m]);
    }
    // slots 0 and L/2 of a packed line: two real modes each (operators are real on them)
    if (cx.first_wave) {
        const Four f = self_eval(cx, [&](const Self& e) {
            if constexpr (GEN)
                return eval_op<true>(op, e.q).x;
            else
                return horner(poly, e.q.q2);
        });
        if (cx.pair_lane) pair_scale(f, v, d[0], d[P / 2]);
    }
#pragma unroll
    for (int m = 0; m < P; ++m) add_to(acc, target, m, d[m]);
}

// Fourier value of an intermediate field at the slots of one line, from the
// dynamic fields' values s there (Sec. "Writing models"):
//   psi = sum_k op_k(q) phi_{src_k} / (1 - L_psi(q)).
// On a packed line the pair slots come out in the same form as the state's:
// (value of the kx = 0 mode, value of the kx = -Nx/2 mode), both real, since
// every operator is real on those four self-conjugate modes.
template <int P, int NF, bool LANES>
__device__ __forceinline__ void interm_line(const DevInterm& I, const float2 (&s)[NF][P], const LineCtx<P, LANES>& cx,
                                            const ModeQ (&q)[P], float2 (&v)[P]) {
    float2 plo = make_float2(0.f, 0.f), phi = make_float2(0.f, 0.f);
#pragma unroll
    for (int m = 0; m < P; ++m) v[m] = make_float2(0.f, 0.f);
    for (int k = 0; k < I.nsrc; ++k) {
        const int src = I.src[k];
        float2 M[P], a[P];
        eval_op_p(I.op[k], cx.q2, q, M);
#pragma unroll
        for (int m = 0; m < P; ++m) {
            a[m] = pick(s, src, m);
            v[m] = cadd(v[m], cmul(M[m], a[m]));
        }
        if (cx.first_wave) {
            const Four f = self_eval(cx, [&](const Self& e) { return eval_op<true>(I.op[k], e.q).x; });
            plo = make_float2(fmaf(f.v[0], a[0].x, plo.x), fmaf(f.v[1], a[0].y, plo.y));
            phi = make_float2(fmaf(f.v[2], a[P / 2].x, phi.x), fmaf(f.v[3], a[P / 2].y, phi.y));
        }
    }
    if (!I.no_den) {  // 1 - L_psi = 1 otherwise
        float2 M[P];
        eval_op_p(I.den, cx.q2, q, M);
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = cmul(v[m], cinv_implicit(1.f, M[m]));
        if (cx.first_wave) {
            const Four f =
                self_eval(cx, [&](const Self& e) { return cinv_implicit(1.f, eval_op<true>(I.den, e.q)).x; });
            plo = make_float2(plo.x * f.v[0], plo.y * f.v[1]);
            phi = make_float2(phi.x * f.v[2], phi.y * f.v[3]);
        }
    }
    if (cx.pair_lane) {
        v[0] = plo;
        v[P / 2] = phi;
    }
}

// the values of factor or linear-term source `src` at the slots of a line:
// a dynamic field's own, or an intermediate's (only plans with the general
// operator code have intermediates)
template <int P, int NF, bool GEN, bool LANES>
__device__ __forceinline__ void source_line(const DevPlan& p, int src, const float2 (&s)[NF][P],
                                            const LineCtx<P, LANES>& cx,
                                            const ModeQ (&qv)[GEN ? P : 1], float2 (&v)[P]) {
    if constexpr (GEN) {
        if (src >= PSS_MAXF) {
            interm_line(p.interm[src - PSS_MAXF], s, cx, qv, v);
            return;
        }
    }
#pragma unroll
    for (int m = 0; m < P; ++m) v[m] = pick(s, src, m);
}

// One block of the update kernel: tile `blk` of lattice `mi`.  In the step
// modes of several lattices (TABLE) the lattice's buffers, counter and flag
// come from the member table and its plan from the plan array (both kernel
// arguments, so the plan reads stay scalar loads).  A launch of one lattice
// (and the transform modes) takes buffers, counter and flag from the
// arguments: its data loads then wait for no table load.
template <int L, int P, int NF, int MODE, int DIM, bool GEN, bool TABLE>
__device__ __forceinline__ void update_block(int mi, int blk, const Member* __restrict__ members,
                                             const DevPlan* __restrict__ plans, const DevPlan* __restrict__ plan_a,
                                             const Bufs& bufs_a, const Geo& geo,
                                             const uint64_t* __restrict__ step_ctr_a, uint32_t* __restrict__ flag_a,
                                             int step_off, const float2* __restrict__ tw_g) {
    using FFT = LineFFT<L, P>;
    constexpr int T = FFT::T;
    extern __shared__ float2 smem[];
    constexpr bool TAB = (MODE == MODE_STEP || MODE == MODE_PROLOGUE) && TABLE;
    const Member* mem = members + mi;  // dereferenced in the step modes only
    // the lattice's plan, buffers and counter: from the tables or from the
    // arguments (selected at compile time, so the unused source is never
    // given an address)
    const DevPlan* pp;
    const Bufs* bp;
    const uint64_t* step_ctr;
    if constexpr (TAB) {
        pp = plans + mi;
        bp = &mem->bufs;
        step_ctr = mem->step_ctr;
    } else {
        pp = plan_a;
        bp = &bufs_a;
        step_ctr = step_ctr_a;
    }
    const DevPlan& p = *pp;
    const Bufs& bufs = *bp;
    const int tc = geo.tc, to = geo.to;
    const int ntile = geo.ntile;
    const int tid = threadIdx.x;
    const int nthr = tc * to * T;
    const int t = tid & (T - 1);
    const int li = tid / T;  // line of the block
    const int cc = li & (tc - 1);
    const int lo = li >> geo.tc_log2;
    const int og = DIM == 2 ? 0 : __builtin_amdgcn_readfirstlane(blk / ntile);  // group of `to` other-index lines
    const int ct = blk - og * ntile;                                            // tile index
    const int o = og * to + lo;
    const int c = ct * tc + cc;  // packed column
    const int nx = geo.nx, ny = geo.ny;
    using I = std::conditional_t<DIM == 2, uint32_t, size_t>;
    const I base = (static_cast<I>(o) * ntile + ct) * L * tc + cc;
    // the exchange arrays: products in, factors (and transform modes' arrays) out
    Exch<I> xin, xout;
    if constexpr (DIM == 2) {
        xin = xout = exch_column(geo, ct, cc, L);
    } else {
        xin = Exch<I>{base, static_cast<I>(tc), false};
        xout = Exch<I>{(static_cast<I>(ct) * ny + o) * tc + cc, static_cast<I>(ntile) * ny * tc, false};
    }
    // this thread's first position and the step from slot to slot
    const I sat = base + static_cast<I>(t) * tc, sstep = static_cast<I>(T) * tc;
    const I iat = xin.at(t), istep = xin.step(T), oat = xout.at(t), ostep = xout.step(T);
    LdsLine ld = FFT::lds_line(smem + li * FFT::kLds);
    // packed-line exchange (the block's first line where it shares that line's
    // block buffer)
    float2* xbuf = FFT::kOne ? smem + FFT::kReg : smem + tc * to * FFT::kLds;
    float2* twl = smem + tc * to * FFT::kLds + fft_xbuf_elems(L, P);
    const int dr = FFT::drev(t);  // gathered / scattered positions dr + m*T
    Twiddles<FFT, L, P> tw;
    // block holds a packed line (block-uniform); this thread is on it
    const bool blk_packed = ct == 0 && (DIM == 2 || og * to == 0 || og * to == (ny >> 1));
    const bool packed = blk_packed && cc == 0 && lo == 0;
    const bool pair_lane = packed && t == 0;  // holds slots 0 and L/2: two real modes each
    // fixed mode indices of a plain line
    int kx_l = c, ky_l = 0;
    if (DIM == 3) {
        ky_l = signed_mode(o, ny);
        if (c == 0 && !packed) {
            if (o < (ny >> 1)) {
                kx_l = 0;
                ky_l = o;
            } else {
                kx_l = -(nx >> 1);
                ky_l = ny - o;
            }
        }
    }

    // packed line only: exchange v (natural order) with the partner slot -u
    // and map it (block-uniform)
    auto exchange = [&](float2 (&v)[P], bool forward) {
        if (!blk_packed) return;
        if constexpr (FFT::kOne) __syncthreads();  // the block buffer's readers are done
        if (packed) {
#pragma unroll
            for (int m = 0; m < P; ++m) xbuf[t + m * T] = v[m];
        }
        __syncthreads();
        if (packed) {
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const int u = t + m * T;
                const float2 b = xbuf[(L - u) & (L - 1)];
                v[m] = forward ? to_slot<L>(u, v[m], b) : from_slot<L>(u, v[m], b);
            }
        }
        __syncthreads();
    };

    if constexpr (MODE == MODE_FWD_STORE) {
        // forward transform of an array in the state layout, stored as the state
        float2 v[P];
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = gload(bufs.in + xin.at(dr + m * T));
        tw.load(tw_g, t, tid, nthr);
        tw.ready(twl, tid, nthr);
        FFT::template dit<-1>(v, ld, t, tw.get());
        exchange(v, true);
#pragma unroll
        for (int m = 0; m < P; ++m) gstore_at<false>(bufs.S[bufs.sel], sat + m * sstep, v[m]);
        return;
    }
    if constexpr (MODE == MODE_INV_OUT) {
        float2 v[P];
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = gload_at(bufs.S[bufs.sel], sat + m * sstep);
        tw.load(tw_g, t, tid, nthr);
        tw.ready(twl, tid, nthr);
        exchange(v, false);
        FFT::template dif<1>(v, ld, t, tw.get());
        if constexpr (FFT::kCross) {
            // a wave of a longer line would write 8 bytes of 64 places far
            // apart: put in order first (4096^2: 56 -> 40 us a launch; the rows
            // of C2R_OUT, gathered 16 bytes a place, gained nothing by it)
            FFT::to_natural(v, ld, t);
#pragma unroll
            for (int m = 0; m < P; ++m) gstore(bufs.out + xout.at(t + m * T), v[m]);
        } else {
#pragma unroll
            for (int m = 0; m < P; ++m) gstore(bufs.out + xout.at(dr + m * T), v[m]);
        }
        return;
    }

    // ---- MODE_STEP, MODE_PROLOGUE or MODE_INTERM_OUT
    // Every read that the step starts from is issued here, before anything
    // waits: the plan's scalars and (plans of one or two fields) its
    // operators as blocks of scalar loads, the first channel, the twiddles
    // and the state.  With the plan read where it is used, the launch spent
    // some 35 scalar-load waits in a row.
    constexpr bool STEP = MODE == MODE_STEP || MODE == MODE_FRAME_STEP;
    constexpr bool HOT = STEP && !GEN && NF <= 2;
    int nf = p.nf, nch = p.nch, ng = p.ng, nd = p.nd;
    float qs[3] = {p.qs[0], p.qs[1], p.qs[2]};
    float dt = p.dt, amp_pair = p.amp_pair, amp_self = p.amp_self;
    uint32_t key0 = p.key0, key1 = p.key1;
    int noisy[NF], fid[NF];
    OpPoly imp[HOT ? NF : 1], noi[HOT ? NF : 1], ch0;
    if constexpr (STEP) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            noisy[f] = p.noisy[f];
            fid[f] = p.fid[f];
        }
    }
    if constexpr (HOT) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            imp[f] = op_poly(p.implicit_op[f]);
            noi[f] = op_poly(p.noise_op[f]);
        }
        ch0 = op_poly(p.ch[0].op[0]);
    }
    const int32_t* lim0 = p.lim[0];
    uint32_t step = 0;
    if constexpr (STEP) step = static_cast<uint32_t>(gload_u64(step_ctr)) + static_cast<uint32_t>(step_off);

    float2 nxt[STEP ? P : 1];
    if constexpr (STEP) {
        // the arrays of a plan without products are null: read the state instead
        const float2* n0 = bufs.N[0] ? bufs.N[0] : bufs.S[0];
#pragma unroll
        for (int m = 0; m < P; ++m) nxt[m] = gload_at(n0, iat + m * istep);
    }
    tw.load(tw_g, t, tid, nthr);
    float2 s[NF][P];  // state, then new state (slot form on a packed line)
    auto load_state = [&]() {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (f == 0 || f < nf) {
#pragma unroll
                for (int m = 0; m < P; ++m) s[f][m] = gload_at(bufs.S[f], sat + m * sstep);
            } else {
#pragma unroll
                for (int m = 0; m < P; ++m) s[f][m] = make_float2(0.f, 0.f);
            }
        }
    };
    // Few points per thread: the launch is a round or two of blocks, and the
    // loads, the noise and the next channel go ahead of what needs them.  With
    // 8 and more points, and in batches, other blocks cover the waits, and what
    // would be held across the transforms costs waves: each is taken where it
    // is used.
    constexpr bool EARLY = P < 8 && !TABLE;
    // 2D lines of 2048 and 4096 and batches also hold nothing across a
    // transform that can be formed after it (addresses, q^2) and draw the noise
    // into the state.  4096: 148 -> 123 registers, two blocks of eight waves
    // per CU instead of one, 91 -> 74 us a launch.  Batches of lines up to
    // 1024: 129 -> 109, four waves a SIMD (64 lattices of 256^2 and 16 of
    // 512^2: 42.8 -> 41.9 us a launch).  In 3D, whose launches are bound by memory, the
    // fourth wave cost more than it hid (256^3: 57 -> 65 us).
    constexpr bool LEAN = STEP && !EARLY && !GEN && DIM == 2;
    if constexpr (MODE == MODE_FRAME_FWD) {
        // the state from real space: the frame was set there
#pragma unroll
        for (int m = 0; m < P; ++m) s[0][m] = gload_at(bufs.in, iat + m * istep);
    } else if constexpr (EARLY || !STEP) {
        load_state();
    }
    if constexpr (STEP) {
        hold(nf), hold(nch), hold(ng), hold(nd), hold(dt), hold(amp_pair), hold(amp_self), hold(key0), hold(key1);
#pragma unroll
        for (int i = 0; i < 3; ++i) hold(qs[i]);
#pragma unroll
        for (int f = 0; f < NF; ++f) hold(noisy[f]), hold(fid[f]);
        hold(step);
    }
    if constexpr (HOT) {
#pragma unroll
        for (int f = 0; f < NF; ++f) hold(imp[f]), hold(noi[f]);
        hold(ch0);
    }
    // the de-aliasing limits of the line for the first factor
    const int kxa = kx_l < 0 ? -kx_l : kx_l, kya = ky_l < 0 ? -ky_l : ky_l;
    const int lrow = kya * ((nx >> 1) + 1);
    int lim_0 = -1, limN_0 = -1;
    if (ng > 0 && ct * tc < geo.ncol[0]) {
        lim_0 = lim0[lrow + kxa];
        if (blk_packed) limN_0 = lim0[lrow + (nx >> 1)];
    }

    const LineModes lmode = line_modes<L, DIM>(nx, ny, qs, packed, kx_l, ky_l);
    // per-slot modes of the line (slot form on a packed line)
    constexpr bool LANES = T >= 4;
    LineCtx<P, LANES> cx;
    auto set_q2 = [&]() {
        int tq = t;
        if constexpr (LEAN) fresh(tq);
#pragma unroll
        for (int m = 0; m < P; ++m) {
            uint32_t lin, lneg;
            slot_at<L>(lmode, tq + m * T, cx.q2[m], lin, lneg);
        }
    };
    if constexpr (!LEAN) set_q2();
    cx.pair_lane = pair_lane;
    cx.first_wave = blk_packed && tid < 64;
    if (cx.first_wave) {
#pragma unroll
        for (int j = 0; j < (LANES ? 1 : 4); ++j)
            cx.self[j] = self_modes<L, DIM>(nx, ny, geo.nz, qs, DIM == 3 ? signed_mode(og * to, ny) : 0,
                                            LANES ? tid : j);
    }
    // general operators: the mode vectors of the slots, once per line
    ModeQ qv[GEN ? P : 1];
    if constexpr (GEN) {
#pragma unroll
        for (int m = 0; m < P; ++m) qv[m] = slot_q<L, DIM>(nx, ny, geo.nz, qs, lmode, t + m * T);
    }

    if constexpr (MODE == MODE_INTERM_OUT) {
        // an intermediate field from the current state, inverse-transformed
        // along the line into `out` (natural order, as MODE_INV_OUT)
        tw.ready(twl, tid, nthr);
        float2 v[P];
        source_line<P, NF, GEN, (T >= 4)>(p, PSS_MAXF + bufs.sel, s, cx, qv, v);
        exchange(v, false);
        FFT::template dif<1>(v, ld, t, tw.get());
#pragma unroll
        for (int m = 0; m < P; ++m) gstore(bufs.out + xout.at(dr + m * T), v[m]);
        return;
    }
    if constexpr (MODE == MODE_PROLOGUE) tw.ready(twl, tid, nthr);
    if constexpr (MODE == MODE_FRAME_FWD) {
        tw.ready(twl, tid, nthr);
        FFT::template dit<-1>(s[0], ld, t, tw.get());
        exchange(s[0], true);
#pragma unroll
        for (int m = 0; m < P; ++m) gstore_at<true>(bufs.S[0], sat + m * sstep, s[0][m]);
    }
    if constexpr (STEP) {
        // The step's noise depends on the step and the modes only.  Per field:
        // of the slots, and of the four self-conjugate modes.
        auto noise_modes = [&](auto FF, auto&& use, Four& e4) {
            constexpr int f = decltype(FF)::value;
            {
                const NoiseKey nk{key0, key1, step, fid[f], amp_pair, amp_self};
                float Dn[P];
                if constexpr (HOT) {
                    horner_p(noi[f], cx.q2, Dn);
                } else if constexpr (GEN) {
                    float2 D2[P];
                    eval_op_p(p.noise_op[f], cx.q2, qv, D2);
#pragma unroll
                    for (int m = 0; m < P; ++m) Dn[m] = D2[m].x;
                } else {
                    horner_p(p.noise_op[f], cx.q2, Dn);
                }
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    float q2m;
                    uint32_t lin, lneg;
                    slot_at<L>(lmode, t + m * T, q2m, lin, lneg);
                    use(m, noise_value<true>(nk, lin, lneg, Dn[m]));
                    // two modes at a time: eight interleaved generators would
                    // hold some fifty registers
                    if ((P >= 8 || LEAN) && (m & 1)) __builtin_amdgcn_sched_barrier(0);
                }
                if (cx.first_wave) {
                    e4 = self_eval(cx, [&](const Self& e) {
                        float Ds;
                        if constexpr (HOT)
                            Ds = horner(noi[f], e.q.q2);
                        else
                            Ds = eval_op<GEN>(p.noise_op[f], e.q).x;
                        return noise_value(nk, e.lin, e.lneg, Ds).x;
                    });
                }
            }
        };
        auto noise_of = [&](auto FF, float2 (&e)[P], Four& e4) {
            constexpr int f = decltype(FF)::value;
            if (f < nf && noisy[f] != 0) {
                noise_modes(FF, [&](int m, float2 v) { e[m] = v; }, e4);
            } else {
#pragma unroll
                for (int m = 0; m < P; ++m) e[m] = make_float2(0.f, 0.f);
            }
        };
        float2 eta[EARLY ? NF : 1][P];
        Four eta4[EARLY ? NF : 1];
        if constexpr (EARLY) {
            static_for<NF>([&](auto FF) { noise_of(FF, eta[decltype(FF)::value], eta4[decltype(FF)::value]); });
        }
        tw.ready(twl, tid, nthr);
        float2 acc[NF][P];  // explicit contributions
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int m = 0; m < P; ++m) acc[f][m] = make_float2(0.f, 0.f);
        // explicit real-space channels: forward transform, then M(q) per mode
        for (int ch = 0; ch < nch; ++ch) {
            const DevChannel& C = p.ch[ch];
            float2 v[P];
#pragma unroll
            for (int m = 0; m < P; ++m) v[m] = nxt[m];
            // each output: its operator times the transform, into its field
            // (one field: one output, so the loop is left out)
            const int nout = NF == 1 ? 1 : C.nout;
            auto load_next = [&]() {
                if (ch + 1 < nch) {
                    auto at = iat;
                    if constexpr (LEAN) fresh(at);
#pragma unroll
                    for (int m = 0; m < P; ++m) nxt[m] = gload_at(bufs.N[ch + 1], at + m * istep);
                }
            };
            if constexpr (EARLY) load_next();
            FFT::template dit<-1>(v, ld, t, tw.get());
            exchange(v, true);
            if constexpr (LEAN) set_q2();
            for (int o2 = 0; o2 < nout; ++o2) {
                const DevOp& op = C.op[o2];
                const int tg = NF == 1 ? 0 : C.target[o2];
                OpPoly poly;
                if constexpr (HOT) {
                    if (ch == 0 && o2 == 0)
                        poly = ch0;
                    else
                        poly = op_poly(op);
                } else if constexpr (!GEN) {
                    poly = op_poly(op);
                }
                accumulate<GEN>(acc, tg, v, op, poly, cx, qv);
            }
            if constexpr (!EARLY) load_next();
        }
        if constexpr (!EARLY) load_state();
        if constexpr (LEAN) set_q2();
        // Fourier-space terms with a single linear factor
        for (int d = 0; d < nd; ++d) {
            const DevDirect& Dd = p.direct[d];
            float2 src[P];  // from the step-n state (an intermediate: its step-n value)
            source_line<P, NF, GEN, (T >= 4)>(p, Dd.src, s, cx, qv, src);
            OpPoly poly;
            if constexpr (!GEN) poly = op_poly(Dd.op);
            accumulate<GEN>(acc, Dd.target, src, Dd.op, poly, cx, qv);
        }
        // semi-implicit update (eq:timeupdate) with in-register noise
        // fields unrolled by template: a loop that the compiler leaves rolled
        // (the general-operator bodies are large) indexes s and acc at run
        // time, which moves both arrays to scratch memory
        uint32_t bad = 0;
        // the new state replaces the old one, or (one field) goes to `out`
        float2* sout[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) sout[f] = bufs.S[f];
        if constexpr (NF == 1 && MODE == MODE_STEP && !TABLE) sout[0] = bufs.out ? bufs.out : bufs.S[0];
        static_for<NF>([&](auto FF) {
            constexpr int f = decltype(FF)::value;
            if (f >= nf) return;
            const bool nz = noisy[f] != 0;
            constexpr int fe = EARLY ? f : 0;
            if constexpr (!EARLY && !LEAN) noise_of(FF, eta[0], eta4[0]);
            if constexpr (LEAN) {
                // two arrays instead of three while the noise is drawn
#pragma unroll
                for (int m = 0; m < P; ++m) s[f][m] = cadd(s[f][m], cscale(acc[f][m], dt));
            }
            const float2 old0 = s[f][0], oldh = s[f][P / 2];
            auto with_acc = [&](float2 v, int m) { return LEAN ? v : cadd(v, cscale(acc[f][m], dt)); };
            if constexpr (LEAN) {
                if (nz) noise_modes(FF, [&](int m, float2 e) { s[f][m] = cadd(s[f][m], e); }, eta4[0]);
            }
            if constexpr (GEN) {
                float2 A[P];
                eval_op_p(p.implicit_op[f], cx.q2, qv, A);
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    float2 r = with_acc(s[f][m], m);
                    if (!LEAN && nz) r = cadd(r, eta[fe][m]);
                    s[f][m] = cmul(r, cinv_implicit(dt, A[m]));
                }
            } else {
                float A[P];
                if constexpr (HOT)
                    horner_p(imp[f], cx.q2, A);
                else
                    horner_p(p.implicit_op[f], cx.q2, A);
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    float2 r = with_acc(s[f][m], m);
                    if (!LEAN && nz) r = cadd(r, eta[fe][m]);
                    s[f][m] = cscale(r, __builtin_amdgcn_rcpf(fmaf(-dt, A[m], 1.f)));
                }
            }
            if (cx.first_wave) {
                const Four inv = self_eval(cx, [&](const Self& e) {
                    float A;
                    if constexpr (HOT)
                        A = horner(imp[f], e.q.q2);
                    else
                        A = eval_op<GEN>(p.implicit_op[f], e.q).x;
                    return cinv_implicit(dt, make_float2(A, 0.f)).x;
                });
                if (pair_lane) {
                    // slots 0 and L/2 hold two real modes each
                    float2 r = with_acc(old0, 0), rh = with_acc(oldh, P / 2);
                    if (nz) {
                        r = make_float2(r.x + eta4[fe].v[0], r.y + eta4[fe].v[1]);
                        rh = make_float2(rh.x + eta4[fe].v[2], rh.y + eta4[fe].v[3]);
                    }
                    pair_scale<2>(inv, {r, rh}, s[f][0], s[f][P / 2]);
                }
            }
            // x * 0 is NaN for a NaN or an infinity, and a sum keeps it
            float fin = 0.f;
#pragma unroll
            for (int m = 0; m < P; ++m) {
                if constexpr (MODE == MODE_STEP) gstore_at<!TABLE>(sout[f], sat + m * sstep, s[f][m]);
                fin = fmaf(s[f][m].x, 0.f, fin);
                fin = fmaf(s[f][m].y, 0.f, fin);
            }
            if (fin != 0.f) bad |= 1u << f;  // a NaN or infinity in the new state
        });
        if (bad) {
            if constexpr (TAB) {
                atomicOr(mem->flag, bad);
            } else {
                atomicOr(flag_a, bad);
            }
        }
    }

    if constexpr (MODE == MODE_FRAME_STEP) {
        exchange(s[0], false);
        FFT::template dif<1>(s[0], ld, t, tw.get());
#pragma unroll
        for (int m = 0; m < P; ++m) gstore_at<true>(bufs.out, oat + m * ostep, s[0][m]);
        return;
    }

    // de-aliased inverse transforms of every factor field (eq:cubicexampledealiased)
    for (int g = 0; g < ng; ++g) {
        // whole tile masked: never read (block-uniform)
        if (ct * tc >= geo.ncol[g]) continue;
        // the factor's Fourier values (a dynamic field's new state, or an
        // intermediate computed from it)
        float2 a[P];
        if constexpr (NF == 1 && !GEN) {
#pragma unroll
            for (int m = 0; m < P; ++m) a[m] = s[0][m];
        } else {
            source_line<P, NF, GEN, (T >= 4)>(p, p.gfield[g], s, cx, qv, a);
        }
        // the largest kept w^2 of this line (packed: of each half)
        int lim = lim_0, limN = limN_0;
        if (g > 0) {
            lim = p.lim[g][lrow + kxa];
            if (blk_packed) limN = p.lim[g][lrow + (nx >> 1)];
        }
        float2 v[P];
#pragma unroll
        for (int m = 0; m < P; ++m) {
            const int u = t + m * T;
            const bool upper = packed && u > (L >> 1);
            const int w = packed ? (upper ? L - u : u) : (u < (L >> 1) ? u : u - L);
            v[m] = w * w <= (upper ? limN : lim) ? a[m] : make_float2(0.f, 0.f);
        }
        if (pair_lane) {
            // slots 0 and L/2: kx = 0 (re) and kx = -Nx/2 (im) at w = 0, -L/2
            const int wh = (L >> 1) * (L >> 1);
            const float2 a0 = a[0], ah = a[P / 2];
            v[0] = make_float2(0 <= lim ? a0.x : 0.f, 0 <= limN ? a0.y : 0.f);
            v[P / 2] = make_float2(wh <= lim ? ah.x : 0.f, wh <= limN ? ah.y : 0.f);
        }
        exchange(v, false);
        FFT::template dif<1>(v, ld, t, tw.get());
        auto at = oat;
        if constexpr (LEAN) fresh(at);
#pragma unroll
        for (int m = 0; m < P; ++m) gstore_at<!TABLE>(bufs.V[g], at + m * ostep, v[m]);
    }
}

template <int L, int P, int NF, int MODE, int DIM, bool GEN, bool TABLE>
__global__ void __launch_bounds__(line_block(L, P)) update_kernel(const Member* __restrict__ members,
                                                      const DevPlan* __restrict__ plans,
                                                      const DevPlan* __restrict__ plan_a, Bufs bufs_a, Geo geo,
                                                      const uint64_t* __restrict__ step_ctr_a,
                                                      uint32_t* __restrict__ flag_a, int step_off,
                                                      const float2* __restrict__ tw_g) {
    // lattice blockIdx.y, XCD-ordered over the whole grid
    const int nb = gridDim.x;
    const int lin_b = TABLE ? xcd_block(blockIdx.y * nb + blockIdx.x, nb * gridDim.y) : xcd_block(blockIdx.x, nb);
    const int mi = TABLE ? __builtin_amdgcn_readfirstlane(lin_b / nb) : 0;
    update_block<L, P, NF, MODE, DIM, GEN, TABLE>(mi, lin_b - mi * nb, members, plans, plan_a, bufs_a, geo,
                                                  step_ctr_a, flag_a, step_off, tw_g);
}

// ------------------------------------------------------ adjoint column kernel
// One reverse step of 2D Model B along y lines (AdjArgs).  Same block shape,
// slot form and LDS layout as the 2D update kernel: TC column lines per
// block, the T threads of a line consecutive, thread t holds slots
// u = t + m*T.  Inner products over all modes become sums over the stored
// slots with weight 2 (a mode and its conjugate), and weight 1 for each real
// component of the pair slots.
//
// 256^2 is latency from end to end: as in the update kernel, every read is
// issued at the top, the noise is formed meanwhile, the limits of the mask
// come from the table and the self-conjugate modes are evaluated in four
// lanes.  14.2 -> 8.2 us a launch.
template <int L, int P, int MODE>
__global__ void __launch_bounds__(line_block(L, P)) adjcol_kernel(AdjArgs aa, Geo geo, const float2* __restrict__ tw_g) {
    using FFT = LineFFT<L, P>;
    constexpr int T = FFT::T;
    constexpr bool LANES = T >= 4;
    extern __shared__ float2 smem[];
    const DevPlan& p = *aa.plan;
    const int tc = geo.tc;
    const int tid = threadIdx.x;
    const int nthr = tc * T;
    const int t = tid & (T - 1);
    const int cc = tid / T;
    const int ct = xcd_block(blockIdx.x, gridDim.x);
    const int c = ct * tc + cc;
    const int nx = geo.nx;
    const uint32_t sat = static_cast<uint32_t>((ct * L + t) * tc + cc), sstep = static_cast<uint32_t>(T * tc);
    const Exch<uint32_t> xch = exch_column(geo, ct, cc, L);
    const uint32_t xat = xch.at(t), xstep = xch.step(T);
    LdsLine ld = FFT::lds_line(smem + cc * FFT::kLds);
    float2* xbuf = FFT::kOne ? smem + FFT::kReg : smem + tc * FFT::kLds;
    float2* twl = smem + tc * FFT::kLds + fft_xbuf_elems(L, P);
    const bool blk_packed = ct == 0;
    const bool packed = blk_packed && cc == 0;
    const bool pair_lane = packed && t == 0, first_wave = blk_packed && tid < 64;
    auto pair_slot = [&](int m) { return pair_lane && (m == 0 || m == P / 2); };

    float qs[3] = {p.qs[0], p.qs[1], p.qs[2]};
    float dt = p.dt, inv_n = p.inv_n, amp_pair = p.amp_pair, amp_self = p.amp_self;
    uint32_t key0 = p.key0, key1 = p.key1;
    int noisy = p.noisy[0], fid = p.fid[0];
    OpPoly noi = op_poly(p.noise_op[0]);
    const int32_t* lim_g = p.lim[0];
    double* const slot = aa.acc + static_cast<size_t>(blockIdx.x) * 3;
    double old[3] = {0.0, 0.0, 0.0};
    if (MODE == MODE_ADJCOL && tid == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) old[i] = slot[i];
    }
    float2 g[P], rin[P], f1[P], f0[P];
    Twiddles<FFT, L, P> tw;
    if (aa.first) {
#pragma unroll
        for (int m = 0; m < P; ++m) g[m] = gload_at(aa.G, sat + m * sstep);
    } else {
#pragma unroll
        for (int m = 0; m < P; ++m) g[m] = gload_at(aa.X, xat + m * xstep);
#pragma unroll
        for (int m = 0; m < P; ++m) rin[m] = gload_at(aa.Rin, sat + m * sstep);
    }
    tw.load(tw_g, t, tid, nthr);
    if constexpr (MODE == MODE_ADJCOL) {
#pragma unroll
        for (int m = 0; m < P; ++m) f1[m] = gload_at(aa.phi1, sat + m * sstep);
#pragma unroll
        for (int m = 0; m < P; ++m) f0[m] = gload_at(aa.phi0, sat + m * sstep);
    }
    hold(dt), hold(inv_n), hold(amp_pair), hold(amp_self), hold(key0), hold(key1), hold(noisy), hold(fid), hold(noi);
#pragma unroll
    for (int i = 0; i < 3; ++i) hold(qs[i]);
    const int lim = lim_g[c];
    const int limN = blk_packed ? lim_g[nx >> 1] : -1;

    auto exchange = [&](float2 (&v)[P], bool forward) {  // as in the update kernel
        if (!blk_packed) return;
        if constexpr (FFT::kOne) __syncthreads();  // the block buffer's readers are done
        if (packed) {
#pragma unroll
            for (int m = 0; m < P; ++m) xbuf[t + m * T] = v[m];
        }
        __syncthreads();
        if (packed) {
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const int u = t + m * T;
                const float2 b = xbuf[(L - u) & (L - 1)];
                v[m] = forward ? to_slot<L>(u, v[m], b) : from_slot<L>(u, v[m], b);
            }
        }
        __syncthreads();
    };
    // the de-aliased values of a line (slot form on the packed line)
    auto masked = [&](float2 (&v)[P]) {
        const float2 a0 = v[0], ah = v[P / 2];
#pragma unroll
        for (int m = 0; m < P; ++m) {
            const int u = t + m * T;
            const bool upper = packed && u > (L >> 1);
            const int w = packed ? (upper ? L - u : u) : (u < (L >> 1) ? u : u - L);
            if (w * w > (upper ? limN : lim)) v[m] = make_float2(0.f, 0.f);
        }
        if (pair_lane) {
            const int wh = (L >> 1) * (L >> 1);
            v[0] = make_float2(0 <= lim ? a0.x : 0.f, 0 <= limN ? a0.y : 0.f);
            v[P / 2] = make_float2(wh <= lim ? ah.x : 0.f, wh <= limN ? ah.y : 0.f);
        }
    };
    const LineModes lmode = line_modes<L, 2>(nx, L, qs, packed, c, 0);
    Self self[LANES ? 1 : 4];
    if (first_wave) {
#pragma unroll
        for (int j = 0; j < (LANES ? 1 : 4); ++j) self[j] = self_modes<L, 2>(nx, L, 1, qs, 0, LANES ? tid : j);
    }
    // the forward step's noise, while the loads above are in flight
    float q2[P];
    float2 eta[P];
    float eta_s[LANES ? 1 : 4];
    {
        const NoiseKey nk{key0, key1, aa.step, fid, amp_pair, amp_self};
        uint32_t lin[P], lneg[P];
        float D[P];
#pragma unroll
        for (int m = 0; m < P; ++m) slot_at<L>(lmode, t + m * T, q2[m], lin[m], lneg[m]);
        if (MODE == MODE_ADJCOL && noisy) {
            horner_p(noi, q2, D);
#pragma unroll
            for (int m = 0; m < P; ++m) eta[m] = noise_value<true>(nk, lin[m], lneg[m], D[m]);
            if (first_wave) {
#pragma unroll
                for (int j = 0; j < (LANES ? 1 : 4); ++j)
                    eta_s[j] = noise_value(nk, self[j].lin, self[j].lneg, horner(noi, self[j].q.q2)).x;
            }
        }
    }
    tw.ready(twl, tid, nthr);

    // g_{n+1}
    if (!aa.first) {
        FFT::template dit<-1>(g, ld, t, tw.get());
        exchange(g, true);
        masked(g);
#pragma unroll
        for (int m = 0; m < P; ++m) g[m] = cadd(rin[m], cscale(g[m], inv_n * aa.b));
    }
    if constexpr (MODE == MODE_ADJFIN) {
#pragma unroll
        for (int m = 0; m < P; ++m) gstore_at<false>(aa.Rout, sat + m * sstep, g[m]);
        return;
    }

    // r_n = g_{n+1} / A, the coefficient sums, -dt q^2 r_n and m phi_n
    double part[3] = {0.0, 0.0, 0.0};  // d/da, d/dk, <r, eta>
    float2 wr[P];
#pragma unroll
    for (int m = 0; m < P; ++m) {
        const float2 r = cscale(g[m], 1.f / (1.f + dt * q2[m] * (aa.a + aa.k * q2[m])));
        wr[m] = cscale(r, -dt * q2[m]);
        if (!pair_slot(m)) {
            const double re1 = static_cast<double>(r.x) * f1[m].x + static_cast<double>(r.y) * f1[m].y;
            part[0] -= 2.0 * dt * q2[m] * re1;
            part[1] -= 2.0 * dt * static_cast<double>(q2[m]) * q2[m] * re1;
            if (noisy)
                part[2] += 2.0 * (static_cast<double>(r.x) * eta[m].x + static_cast<double>(r.y) * eta[m].y);
            g[m] = r;
        }
    }
    if (first_wave) {
        // the pair slots: four real modes, one per lane (or all in one thread),
        // from the values that the first thread holds
        const float gp[4] = {g[0].x, g[0].y, g[P / 2].x, g[P / 2].y};
        const float fp[4] = {f1[0].x, f1[0].y, f1[P / 2].x, f1[P / 2].y};
        auto mode = [&](float q, float gv, float f1v, float es) {
            const float r = gv / (1.f + dt * q * (aa.a + aa.k * q));
            const double e = static_cast<double>(r) * f1v;
            part[0] -= dt * static_cast<double>(q) * e;
            part[1] -= dt * static_cast<double>(q) * q * e;
            if (noisy) part[2] += static_cast<double>(r) * es;
            return r;
        };
        Four r, q;
        if constexpr (LANES) {
            float gl = 0.f, fl = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gp[j]), 0));
                const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fp[j]), 0));
                gl = (tid & 3) == j ? a : gl;
                fl = (tid & 3) == j ? b : fl;
            }
            const double keep[3] = {part[0], part[1], part[2]};
            const float rl = mode(self[0].q.q2, gl, fl, eta_s[0]);
            if (tid >= 4) {  // lanes 0 to 3 add the four modes once
#pragma unroll
                for (int i = 0; i < 3; ++i) part[i] = keep[i];
            }
            r = four_lanes(rl);
            q = four_lanes(self[0].q.q2);
        } else if (pair_lane) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                q.v[j] = self[j].q.q2;
                r.v[j] = mode(q.v[j], gp[j], fp[j], eta_s[j]);
            }
        }
        if (pair_lane) {
            g[0] = make_float2(r.v[0], r.v[1]);
            g[P / 2] = make_float2(r.v[2], r.v[3]);
            wr[0] = make_float2(-dt * q.v[0] * r.v[0], -dt * q.v[1] * r.v[1]);
            wr[P / 2] = make_float2(-dt * q.v[2] * r.v[2], -dt * q.v[3] * r.v[3]);
        }
    }
#pragma unroll
    for (int m = 0; m < P; ++m) gstore_at<false>(aa.Rout, sat + m * sstep, g[m]);
    exchange(wr, false);
    FFT::template dif<1>(wr, ld, t, tw.get());
#pragma unroll
    for (int m = 0; m < P; ++m) gstore_at<false>(aa.W, xat + m * xstep, wr[m]);
    masked(f0);
    exchange(f0, false);
    FFT::template dif<1>(f0, ld, t, tw.get());
#pragma unroll
    for (int m = 0; m < P; ++m) gstore_at<false>(aa.U, xat + m * xstep, f0[m]);
    if (aa.D > 0.f) part[2] /= 2.0 * aa.D;
    block_sum_to_slot(part, old, slot);
}

#if defined(PSS_COMMON)
// terminal seed of the adjoint: g(k) = coef[shell(k)] phi(k) on the 2D packed
// state layout (slot form on column 0), shell(k) = rint(|k|)
__global__ void adjseed_kernel(const float2* __restrict__ phi, float2* __restrict__ g, const float* __restrict__ coef,
                               int nshell, int nx, int ny, int tc) {
    const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t total = static_cast<int64_t>(nx / 2) * ny;
    if (e >= total) return;
    const int cc = static_cast<int>(e % tc);
    const int y = static_cast<int>((e / tc) % ny);
    const int col = static_cast<int>(e / (static_cast<int64_t>(tc) * ny)) * tc + cc;
    auto cf = [&](int kx, int ky) {
        const int j = static_cast<int>(rintf(sqrtf(static_cast<float>(kx * kx + ky * ky))));
        return (j >= 1 && j < nshell) ? coef[j] : 0.f;
    };
    const float2 v = phi[e];
    float2 o;
    if (col > 0) {
        const float s = cf(col, y < ny / 2 ? y : y - ny);
        o = make_float2(s * v.x, s * v.y);
    } else if (y == 0 || y == ny / 2) {
        const int w = y == 0 ? 0 : -(ny / 2);
        o = make_float2(cf(0, w) * v.x, cf(-(nx / 2), w) * v.y);
    } else if (y < ny / 2) {
        const float s = cf(0, y);
        o = make_float2(s * v.x, s * v.y);
    } else {
        const float s = cf(-(nx / 2), ny - y);
        o = make_float2(s * v.x, s * v.y);
    }
    g[e] = o;
}
#endif  // PSS_COMMON

// ----------------------------------------------------------------- y pass
// 3D only: lines along y for fixed (c, z); block = TC columns x TZ values of
// z, the T threads of a line consecutive.  Input [z][ctile][y][TC].  The
// inverse pass writes the same layout, the forward pass writes the state
// layout [y][ctile][z][TC].
//
// Column 0 arrives from the x pass as X(0) + i X(Nx/2), both real; after the
// forward y transform it is Y(ky) = Y0(ky) + i YN(ky) with Y0, YN Hermitian
// in ky.  The forward pass re-packs it so that every z line of column 0
// except ky = 0, Ny/2 holds single modes:
//   slot ky in (0, Ny/2)   : Y0(ky)          (modes kx = 0)
//   slot Ny-ky             : YN(ky)          (modes kx = Nx/2)
//   slots 0 and Ny/2       : Y unchanged     (packed, Hermitian along z)
// and the inverse pass undoes it before transforming.
template <int L, int P, int MODE>
__global__ void __launch_bounds__(line_block(L, P)) ypass_kernel(YArgs ya, Geo geo, const float2* __restrict__ tw_g) {
    using FFT = LineFFT<L, P>;
    constexpr int T = FFT::T;
    extern __shared__ float2 smem[];
    const int tc = geo.tc, tz = geo.tz;
    const int ntile = geo.ntile;
    const int nz = geo.nz;
    const int tid = threadIdx.x;
    const int nthr = tc * tz * T;
    const int t = tid & (T - 1);
    const int li = tid / T;
    const int cc = li & (tc - 1);
    const int lz = li >> geo.tc_log2;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int ct = blk % ntile;
    const int z = (blk / ntile) * tz + lz;
    const int c = ct * tc + cc;
    LdsLine ld = FFT::lds_line(smem + li * FFT::kLds);
    float2* xb = smem + tc * tz * FFT::kLds + lz * L;  // column-0 exchange, one line per z
    const int dr = FFT::drev(t);
    Twiddles<FFT, L, P> tw;
    tw.load(tw_g, t, tid, nthr);
    tw.ready(smem + tc * tz * FFT::kLds + tz * L, tid, nthr);
    const size_t ibase = (static_cast<size_t>(z) * ntile + ct) * L * tc + cc;
    const size_t obase = MODE == MODE_YFWD ? (static_cast<size_t>(ct) * nz + z) * tc + cc : ibase;
    const size_t ostride = MODE == MODE_YFWD ? static_cast<size_t>(ntile) * nz * tc : static_cast<size_t>(tc);

    for (int a = 0; a < ya.n; ++a) {
        if (ct * tc >= ya.ncol[a]) continue;  // tile holds no kept column (block-uniform)
        const float2* __restrict__ src = ya.src[a];
        float2* __restrict__ dst = ya.dst[a];
        float2 v[P];
        if constexpr (MODE == MODE_YINV) {
            // gathered at the digit-reversed positions, natural order out
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const int y = dr + m * T;
                const float2 s1 = src[ibase + y * tc];
                if (c == 0 && y != 0 && y != (L >> 1)) {
                    const float2 s2 = src[ibase + (L - y) * tc];
                    v[m] = y < (L >> 1) ? make_float2(s1.x - s2.y, s1.y + s2.x)   // Y0 + i YN
                                        : make_float2(s2.x + s1.y, s1.x - s2.y);  // conj(Y0) + i conj(YN)
                } else {
                    v[m] = s1;
                }
            }
            // in place (src == dst) is safe: a line is read whole before any of
            // it is written, within one wave or across the transform's barrier
            FFT::template dit<1>(v, ld, t, tw.get());
#pragma unroll
            for (int m = 0; m < P; ++m) dst[obase + (t + m * T) * ostride] = v[m];
        } else {
#pragma unroll
            for (int m = 0; m < P; ++m) v[m] = src[ibase + (t + m * T) * tc];
            FFT::template dif<-1>(v, ld, t, tw.get());
            if (ct == 0) {
                // column 0: the partner of ky is L - ky, exchanged by natural position
                if (c == 0) {
#pragma unroll
                    for (int m = 0; m < P; ++m) xb[dr + m * T] = v[m];
                }
                __syncthreads();
                if (c == 0) {
#pragma unroll
                    for (int m = 0; m < P; ++m) {
                        const int y = dr + m * T;
                        if (y == 0 || y == (L >> 1)) continue;
                        const float2 a0 = v[m], b0 = xb[L - y];
                        v[m] = y < (L >> 1) ? make_float2(0.5f * (a0.x + b0.x), 0.5f * (a0.y - b0.y))   // Y0(y)
                                            : make_float2(0.5f * (a0.y + b0.y), 0.5f * (a0.x - b0.x));  // YN(L-y)
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int m = 0; m < P; ++m) dst[obase + (dr + m * T) * ostride] = v[m];
        }
    }
}

// ----------------------------------------------------------------- x kernel
// 1024^2: the launch was bound by its gather (16 bytes of each 128-byte line
// of [c][y] columns, in digit-reversed order: one line a lane, 1.4 us), by
// the loops over factor powers and by scalar-load waits; with grouped rows,
// natural order and straight-line powers 8.2 -> 6.7 us, KPZ 11.6 -> 7.6 us,
// Model H 31 -> 18 us.
// What is left is memory latency (1.2 us), two transforms and the launch.
// Rows of length L = Nx; block = RB consecutive rows, pair pr = rows
// (2 pr, 2 pr + 1) packed as one complex line held by T consecutive threads.
// Packed-column arrays are read and written in whole tile blocks of RB*TC
// contiguous elements.
// a[m] *= z[m]^n by components, n <= 8 uniform: one forward branch out of a
// straight line instead of a loop
template <int E, int P>
__device__ __forceinline__ void times_power(float2 (&a)[P], const float2 (&z)[P], int n) {
    if constexpr (E < PSS_MAXPOW) {
        if (n <= E) return;
#pragma unroll
        for (int m = 0; m < P; ++m) {
            a[m].x *= z[m].x;
            a[m].y *= z[m].y;
        }
        times_power<E + 1>(a, z, n);
    }
}

// One block of the x kernel: row block `blk` of lattice `mi` (as in the update kernel)
template <int L, int P, int NG, int MODE, bool TABLE>
__device__ __forceinline__ void xrow_block(int mi, int blk, const Member* __restrict__ members,
                                           const DevPlan* __restrict__ plans, const DevPlan* __restrict__ plan_a,
                                           const Bufs& bufs_a, const Geo& geo, const float2* __restrict__ tw_g,
                                           int64_t advance, uint64_t* __restrict__ step_ctr_a) {
    using FFT = LineFFT<L, P>;
    constexpr int T = FFT::T;
    constexpr int NC = L / 2;  // packed columns
    extern __shared__ float2 smem[];
    constexpr bool TAB = MODE == MODE_STEP && TABLE;  // as in the update kernel
    const Member* mem = members + mi;
    const DevPlan* pp;
    const Bufs* bp;
    if constexpr (TAB) {
        pp = plans + mi;
        bp = &mem->bufs;
    } else {
        pp = plan_a;
        bp = &bufs_a;
    }
    const DevPlan& p = *pp;
    const Bufs& bufs = *bp;
    const int tc = geo.tc, rb = geo.rb;
    const int ntile = NC / tc;
    const int tid = threadIdx.x;
    const int nthr = (rb >> 1) * T;
    const int pr = tid / T;  // pair within the block
    const int t = tid & (T - 1);
    const int r0 = blk * rb;  // first row; row index = z*Ny + y
    const int ny = geo.ny;
    const int zr = geo.nz == 1 ? 0 : r0 / ny;  // z of the block (0 in 2D)
    const int y0 = r0 - zr * ny;     // first y of the block
    const int lt = geo.tc_log2;
    LdsLine ld = FFT::lds_line(smem + pr * FFT::kLds);
    const int dr = FFT::drev(t);
    Twiddles<FFT, L, P> tw;
    float2* const twl = smem + (rb >> 1) * FFT::kLds;

    // Gather the packed complex input Z[k] = X_row0[k] + i X_row1[k] of pair
    // pr at k = k0 + m T straight from the packed-column array (columns
    // [0, ncol) are stored; the others are zero); all loads are issued together.
    // A step gathers in natural order (k0 = t: neighbouring threads read
    // neighbouring columns), transforms to digit-reversed x, where the
    // products do not mind the order, and back to natural k; the modes that
    // deliver or take real rows need natural x and gather at k0 = D(t).
    const int yr = y0 + 2 * pr;  // the pair's first row in its plane
    const size_t row0 = geo.grp ? (static_cast<size_t>(yr >> 2) * ntile << 2) + (yr & 3)
                                : (static_cast<size_t>(zr) * ntile * ny + yr) * tc;
    const size_t tstride = geo.grp ? 4 : static_cast<size_t>(ny) * tc;  // one column tile
    auto build_z = [&](float2 (&v)[P], const float2* __restrict__ src, int ncol, int k0) {
        // all loads first, without control flow between them; a dropped
        // column reads column 0 and then counts as zero
        float2 a[P], b[P];
        if (tc == 1) {
            // one-column tiles: the pair's two rows are neighbours, and the
            // row pair starts at an even row, so one aligned 16-byte load
            // takes both (half the address work of two 8-byte loads)
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const int k = k0 + m * T;
                const int kk = (k == NC) ? 0 : (k < NC ? k : L - k);
                const int kc = kk < ncol ? kk : 0;
                gload_pair(src + row0 + kc * tstride, a[m], b[m]);
            }
        } else {
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const int k = k0 + m * T;
                const int kk = (k == NC) ? 0 : (k < NC ? k : L - k);
                const int kc = kk < ncol ? kk : 0;
                const size_t off = row0 + (kc >> lt) * tstride + (kc & (tc - 1));
                a[m] = gload(src + off);
                b[m] = gload(src + off + tc);
            }
        }
#pragma unroll
        for (int m = 0; m < P; ++m) {
            const int k = k0 + m * T;
            const int kk = (k == NC) ? 0 : (k < NC ? k : L - k);
            const float2 zero = make_float2(0.f, 0.f);
            const float2 am = kk < ncol ? a[m] : zero, bm = kk < ncol ? b[m] : zero;
            float2 z;
            if (k == 0) {
                z = make_float2(am.x, bm.x);
            } else if (k == NC) {
                z = make_float2(am.y, bm.y);
            } else {
                z = k < NC ? make_float2(am.x - bm.y, am.y + bm.x) : make_float2(am.x + bm.y, bm.x - am.y);
            }
            v[m] = z;
        }
    };
    // Stage the forward transform W (held at k = k0 + m T) of every pair in
    // LDS at its natural positions, then unpack the two real rows of each
    // pair and store whole packed-column tiles.  A line wider than a wave
    // stages in its next block buffer; a narrower one in its own region
    // (its wave is done with it).  The caller separates consecutive calls by
    // a block barrier when the staging region is the in-wave one.
    auto store_rows = [&](const float2 (&w)[P], float2* __restrict__ dst, int k0) {
        float2* stage = FFT::kCross ? ld.next_blk() : ld.wl;
        if constexpr (!FFT::kCross) wave_lds_sync();  // after the transform's last in-wave reads
        if constexpr (FFT::kOne) __syncthreads();     // the block buffer's readers are done
#pragma unroll
        for (int m = 0; m < P; ++m) stage[k0 + m * T] = w[m];
        __syncthreads();
        if (tc == 1) {
            // one-column tiles: a pair's two rows are neighbours in the
            // column, so one thread unpacks both and stores 16 bytes (half
            // the LDS reads and stores of an element a thread)
            const float2* W = stage;
            float2* const d0 = dst + row0;
#pragma unroll
            for (int j = 0; j < (NC + T - 1) / T; ++j) {
                const int c = t + j * T;
                if (NC % T != 0 && c >= NC) break;
                const float2 a = W[c], b = W[c == 0 ? NC : L - c];
                const float2 lo = c == 0 ? make_float2(a.x, b.x) : make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
                const float2 hi = c == 0 ? make_float2(a.y, b.y) : make_float2(0.5f * (a.y + b.y), 0.5f * (b.x - a.x));
                gstore_pair_sel<!TABLE>(d0 + c * tstride, lo, hi);
            }
            return;
        }
        const int lp = geo.rb_log2 + lt;  // log2(rb * tc)
        const int total = ntile << lp;
        const size_t sbase = (static_cast<size_t>(zr) * ntile) * ny + y0;
#pragma unroll 4
        for (int i = tid; i < total; i += nthr) {
            const int tl = i >> lp, rem = i & ((1 << lp) - 1);
            const int r = rem >> lt, cc = rem & (tc - 1);
            const int c = (tl << lt) + cc;
            const float2* W = smem + (r >> 1) * FFT::kLds + (FFT::kCross ? (stage - ld.wl) : 0);
            const float2 a = W[c], b = W[c == 0 ? NC : L - c];
            float2 o = (r & 1) ? make_float2(0.5f * (a.y + b.y), 0.5f * (b.x - a.x))
                               : make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
            if (c == 0) o = (r & 1) ? make_float2(a.y, b.y) : make_float2(a.x, b.x);
            gstore_sel<!TABLE>(dst + ((sbase + static_cast<size_t>(tl) * ny + r) << lt) + cc, o);
        }
    };

    if constexpr (MODE == MODE_R2C_IN) {
        // real rows -> packed columns (forward transform, unnormalised)
        const float* __restrict__ src = bufs.real_in;
        float2 v[P];
#pragma unroll
        for (int m = 0; m < P; ++m) {
            const int x = t + m * T;
            v[m] = make_float2(src[static_cast<size_t>(r0 + 2 * pr) * L + x],
                               src[static_cast<size_t>(r0 + 2 * pr + 1) * L + x]);
        }
        tw.load(tw_g, t, tid, nthr);
        tw.ready(twl, tid, nthr);
        FFT::template dif<-1>(v, ld, t, tw.get());
        store_rows(v, bufs.out, dr);
        return;
    }
    if constexpr (MODE == MODE_C2R_OUT) {
        float2 v[P];
        build_z(v, bufs.in, NC, dr);
        tw.load(tw_g, t, tid, nthr);
        tw.ready(twl, tid, nthr);
        FFT::template dit<1>(v, ld, t, tw.get());
        float* __restrict__ dst = bufs.real_out;
#pragma unroll
        for (int m = 0; m < P; ++m) {
            const int x = t + m * T;
            dst[static_cast<size_t>(r0 + 2 * pr) * L + x] = v[m].x * p.inv_n;
            dst[static_cast<size_t>(r0 + 2 * pr + 1) * L + x] = v[m].y * p.inv_n;
        }
        return;
    }

    if constexpr (MODE == MODE_FRAME_ROW) {
        // the state's rows to real space, the frame's values on its sites, and
        // back: the row pair is staged in LDS at natural x, where the threads
        // of the pair write the entries of its two rows
        float2 v[P];
        build_z(v, bufs.in, NC, t);
        tw.load(tw_g, t, tid, nthr);
        const int32_t* __restrict__ fr = bufs.frame_rows + yr;
        const int e0 = fr[0], e1 = fr[1], e2 = fr[2];
        float inv_n = p.inv_n;
        hold(inv_n);
        const int2* __restrict__ ent = reinterpret_cast<const int2*>(bufs.frame_rows + ny + 2);
        tw.ready(twl, tid, nthr);
        FFT::template dif<1>(v, ld, t, tw.get());
        float2* stage = FFT::kCross ? ld.next_blk() : ld.wl;
        auto sync = [&]() {
            if constexpr (FFT::kCross) {
                __syncthreads();
            } else {
                wave_lds_sync();
            }
        };
        if constexpr (FFT::kOne || !FFT::kCross) sync();
#pragma unroll
        for (int m = 0; m < P; ++m) stage[dr + m * T] = cscale(v[m], inv_n);
        sync();
        for (int i = e0 + t; i < e2; i += T) {
            const int2 e = ent[i];
            float* w = reinterpret_cast<float*>(stage + e.x);
            w[i < e1 ? 0 : 1] = __int_as_float(e.y);
        }
        sync();
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = stage[dr + m * T];
        FFT::template dit<-1>(v, ld, t, tw.get());
        store_rows(v, bufs.out, t);
        return;
    }

    if constexpr (MODE == MODE_ADJROW) {
        // reverse step, real space: u = F^-1[m phi_n] (rows of V[0], kept
        // columns only), w = N F^-1[-dt q^2 r] (rows of V[1], unnormalised),
        // 3 u^2 w -> forward x transform into N[0] (the column kernel applies
        // the factor b); and the FP64 sum of u^3 w, which is
        // <r, -dt q^2 F[u^3]> = dL/db of the step, by Parseval
        double old[1] = {0.0};
        if (tid == 0) old[0] = bufs.acc[blockIdx.x];
        float2 u[P], w[P];
        build_z(u, bufs.V[0], geo.ncol[0], t);
        build_z(w, bufs.V[1], NC, t);
        tw.load(tw_g, t, tid, nthr);
        tw.ready(twl, tid, nthr);
        FFT::template dif<1>(u, ld, t, tw.get());
        FFT::template dif<1>(w, ld, t, tw.get());
        double part[1] = {0.0};
#pragma unroll
        for (int m = 0; m < P; ++m) {
            const float ux = u[m].x * p.inv_n, uy = u[m].y * p.inv_n;
            part[0] += static_cast<double>(ux) * ux * ux * w[m].x + static_cast<double>(uy) * uy * uy * w[m].y;
            u[m] = make_float2(3.f * ux * ux * w[m].x, 3.f * uy * uy * w[m].y);
        }
        FFT::template dit<-1>(u, ld, t, tw.get());
        store_rows(u, bufs.N[0], t);
        block_sum_to_slot(part, old, bufs.acc + blockIdx.x);
        return;
    }

    // MODE_STEP: the last step of a replayed chunk moves the member's step
    // counter on (no later kernel of the chunk reads it)
    if (advance != 0 && r0 == 0 && tid == 0) {
        if constexpr (TAB) {
            *mem->step_ctr += static_cast<uint64_t>(advance);
        } else {
            *step_ctr_a += static_cast<uint64_t>(advance);
        }
    }
    // the plan's scalars and the first channel's first product as one block of
    // scalar loads ahead of the transforms
    float inv_n = p.inv_n;
    int nch = p.nch, ng = NG > 4 ? p.ng : NG;
    int np0 = p.ch[0].nprod;
    float c0 = p.ch[0].prod[0].coef;
    static_assert(sizeof(p.ch[0].prod[0].pow) == 8, "eight factor slots");
    uint32_t pw0[2];
    __builtin_memcpy(pw0, p.ch[0].prod[0].pow, sizeof(pw0));
    // real-space values of every factor field (the variant with room for
    // more than four holds zeros in the slots beyond the plan's)
    float2 z[NG][P];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (NG > 4 && g >= ng) {
#pragma unroll
            for (int m = 0; m < P; ++m) z[g][m] = make_float2(0.f, 0.f);
            continue;
        }
        float2 v[P];
        build_z(v, bufs.V[g], geo.ncol[g], t);
        if (g == 0) {
            tw.load(tw_g, t, tid, nthr);
            hold(inv_n), hold(nch), hold(ng), hold(np0), hold(c0), hold(pw0[0]), hold(pw0[1]);
            tw.ready(twl, tid, nthr);
        }
        FFT::template dif<1>(v, ld, t, tw.get());
#pragma unroll
        for (int m = 0; m < P; ++m) z[g][m] = cscale(v[m], inv_n);
    }
    // products per channel, forward transform, store
    for (int ch = 0; ch < nch; ++ch) {
        const DevChannel& C = p.ch[ch];
        float2 w[P];
#pragma unroll
        for (int m = 0; m < P; ++m) w[m] = make_float2(0.f, 0.f);
        const int np = ch == 0 ? np0 : C.nprod;
        for (int k = 0; k < np; ++k) {
            // the factor powers read as two words (scalar loads)
            float cf = c0;
            uint32_t pw[2] = {pw0[0], pw0[1]};
            if (ch > 0 || k > 0) {
                const DevProd& pd = C.prod[k];
                cf = pd.coef;
                __builtin_memcpy(pw, pd.pow, sizeof(pw));
            }
            float2 a[P];
#pragma unroll
            for (int m = 0; m < P; ++m) a[m] = make_float2(cf, cf);
            // the powers are uniform: one loop per factor for all points
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int pg = static_cast<int>((pw[g >> 2] >> (8 * (g & 3))) & 0xffu);
                times_power<0>(a, z[g], pg);
            }
#pragma unroll
            for (int m = 0; m < P; ++m) w[m] = cadd(w[m], a[m]);
        }
        if (!FFT::kCross && ch > 0) __syncthreads();  // the previous channel's rows are stored
        FFT::template dit<-1>(w, ld, t, tw.get());
        store_rows(w, bufs.N[ch], t);
    }
}

template <int L, int P, int NG, int MODE, bool TABLE>
__global__ void __launch_bounds__(line_block(L, P)) xrow_kernel(const Member* __restrict__ members,
                                                    const DevPlan* __restrict__ plans,
                                                    const DevPlan* __restrict__ plan_a, Bufs bufs_a, Geo geo,
                                                    const float2* __restrict__ tw_g, int64_t advance,
                                                    uint64_t* __restrict__ step_ctr_a) {
    const int nb = gridDim.x;
    const int lin_b = TABLE ? xcd_block(blockIdx.y * nb + blockIdx.x, nb * gridDim.y) : xcd_block(blockIdx.x, nb);
    const int mi = TABLE ? __builtin_amdgcn_readfirstlane(lin_b / nb) : 0;
    xrow_block<L, P, NG, MODE, TABLE>(mi, lin_b - mi * nb, members, plans, plan_a, bufs_a, geo, tw_g, advance,
                                      step_ctr_a);
}

#if defined(PSS_COMMON)
// ---------------------------------------------------------------- utilities
__global__ void advance_kernel(uint64_t* step_ctr, int64_t k) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *step_ctr += static_cast<uint64_t>(k);
}

__global__ void advance_many_kernel(uint64_t* const* __restrict__ ctrs, int n, int64_t k) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) *ctrs[i] += static_cast<uint64_t>(k);
}

// a boundary frame on a real-space array: site frame[i].x takes the value
// whose bits are frame[i].y
__global__ void apply_frame_kernel(float* __restrict__ real, const int2* __restrict__ frame, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const int2 e = frame[i];
        real[e.x] = __int_as_float(e.y);
    }
}

// read and clear the non-finite flag that follows each member's step counter
__global__ void take_flags_kernel(uint64_t* const* __restrict__ ctrs, int n, uint32_t* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = atomicExch(reinterpret_cast<uint32_t*>(ctrs[i] + 1), 0u);
}

__global__ void init_uniform_kernel(float* __restrict__ out, int64_t n, uint32_t field, uint32_t key0,
                                    uint32_t key1, double lo, double hi) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint4 w = philox4x32_10(make_uint4(static_cast<uint32_t>(i), 0u, field, 1u), key0, key1);
    const double u = (static_cast<double>(w.x >> 9) + 0.5) * 1.1920928955078125e-07;
    out[i] = static_cast<float>(__dadd_rn(lo, __dmul_rn(hi - lo, u)));
}

__global__ void philox_kernel(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                              int64_t count, uint32_t* __restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const uint4 w = philox4x32_10(make_uint4(c0 + static_cast<uint32_t>(i), c1, c2, c3), k0, k1);
    reinterpret_cast<uint4*>(out)[i] = w;
}


// Shell sums for the structure factor.  Thread i handles packed element i of
// the 2D tiled layout [ctile][y][TC]; interior columns stand for the mode and
// its conjugate partner (weight 2); column 0 is unpacked into kx = 0 and
// kx = Nx/2 (weight 1 each) with the partner element at -y.  With dim = 1 the
// array is a full spectrum, element (kz Ny + ky) Nx + kx for mode (kx, ky, kz)
// (weight 1): 1D lines and mixed-radix 2D and 3D lattices.  shell_terms calls
// emit(j, t) for every term t = w * scale * |phi_hat|^2 of shell j.
//
// The sums are exact, so they do not depend on the order in which the
// threads and blocks add: a first pass takes the largest binary exponent E_j
// of the terms of each shell (a max, order-free), a second adds every term
// as the integer round(t * 2^(61 - e_j)) (e_j = E_j - 1023, so each is below
// 2^62) into a 128-bit accumulator (64-bit atomics with carry; integer sums
// are associative), and a last pass turns the integer back into a double.
// Each term is rounded once, to 2^-62 of the shell's largest term.
template <typename F>
__device__ __forceinline__ void shell_terms(const float2* __restrict__ S, int64_t e, int nx, int ny, int nz, int tc,
                                            int dim, int nshell, double scale, F&& emit) {
    auto mag = [](float2 v) { return static_cast<double>(v.x) * v.x + static_cast<double>(v.y) * v.y; };
    auto add = [&](int kx, int ky, int kz, double v, int w) {
        const double kk = static_cast<double>(kx) * kx + static_cast<double>(ky) * ky + static_cast<double>(kz) * kz;
        const int j = static_cast<int>(rint(sqrt(kk)));
        if (j >= 1 && j < nshell) emit(j, scale * v * w, static_cast<unsigned int>(w));
    };
    if (dim == 1) {
        // a full complex spectrum (1D lines, mixed-radix 2D and 3D
        // lattices): each mode once
        const int kx = static_cast<int>(e % nx), ky = static_cast<int>((e / nx) % ny),
                  kz = static_cast<int>(e / (static_cast<int64_t>(nx) * ny));
        add(kx < nx / 2 ? kx : kx - nx, ny == 1 ? 0 : (ky < ny / 2 ? ky : ky - ny),
            nz == 1 ? 0 : (kz < nz / 2 ? kz : kz - nz), mag(S[e]), 1);
        return;
    }
    const int ncols = nx / 2;
    const int ntile = ncols / tc;
    const int cc = static_cast<int>(e % tc);
    const int64_t r = e / tc;
    int c, y, z;
    if (dim == 2) {
        y = static_cast<int>(r % ny);
        c = static_cast<int>(r / ny) * tc + cc;
        z = 0;
    } else {
        z = static_cast<int>(r % nz);
        const int64_t r2 = r / nz;
        c = static_cast<int>(r2 % ntile) * tc + cc;
        y = static_cast<int>(r2 / ntile);
    }
    const int ky = y < ny / 2 ? y : y - ny;
    const int kz = nz == 1 ? 0 : (z < nz / 2 ? z : z - nz);
    const float2 a = S[e];
    if (c > 0) {
        add(c, ky, kz, mag(a), 2);
        return;
    }
    // column 0: slot form along the update axis on packed lines
    const bool packed = dim == 2 || y == 0 || y == ny / 2;
    if (!packed) {
        if (y < ny / 2)
            add(0, y, kz, mag(a), 2);
        else
            add(-(nx / 2), ny - y, kz, mag(a), 2);
        return;
    }
    const int L = dim == 2 ? ny : nz;
    const int u = dim == 2 ? y : z;
    const int ky0 = dim == 2 ? 0 : ky;
    auto at = [&](int w) { return dim == 2 ? make_int2(w, 0) : make_int2(ky0, w); };  // (ky, kz) of index w
    if (u == 0 || u == L / 2) {
        const int w = u == 0 ? 0 : -(L / 2);
        const int2 yz = at(w);
        add(0, yz.x, yz.y, static_cast<double>(a.x) * a.x, 1);
        add(-(nx / 2), yz.x, yz.y, static_cast<double>(a.y) * a.y, 1);
    } else if (u < L / 2) {
        const int2 yz = at(u);
        add(0, yz.x, yz.y, mag(a), 2);
    } else {
        const int2 yz = at(L - u);
        add(-(nx / 2), yz.x, yz.y, mag(a), 2);
    }
}

// order key of a term: twice its biased exponent, +1 for a NaN (so that a
// NaN wins over an infinity, as it would in a plain sum)
__device__ __forceinline__ unsigned int shell_key(double t) {
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(t));
    const unsigned int E = static_cast<unsigned int>((b >> 52) & 0x7ffull);
    const bool nan = E == 0x7ffu && (b & 0xfffffffffffffull) != 0ull;
    return 2u * E + (nan ? 1u : 0u);
}

__device__ __forceinline__ int64_t shell_total(int nx, int ny, int nz, int dim) {
    return dim == 1 ? static_cast<int64_t>(nx) * ny * nz : static_cast<int64_t>(nx / 2) * ny * nz;
}

// pass 1: key[j] = max over the terms of shell j
__global__ void shell_keys_kernel(const float2* __restrict__ S, int nx, int ny, int nz, int tc, int dim, double scale,
                                  int nshell, unsigned int* __restrict__ gkey) {
    extern __shared__ unsigned int lkey[];
    for (int i = threadIdx.x; i < nshell; i += blockDim.x) lkey[i] = 0u;
    __syncthreads();
    const int64_t total = shell_total(nx, ny, nz, dim);
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
         e += static_cast<int64_t>(gridDim.x) * blockDim.x)
        shell_terms(S, e, nx, ny, nz, tc, dim, nshell, scale,
                    [&](int j, double t, unsigned int) { atomicMax(&lkey[j], shell_key(t)); });
    __syncthreads();
    for (int i = threadIdx.x; i < nshell; i += blockDim.x)
        if (lkey[i]) atomicMax(&gkey[i], lkey[i]);
}

// 128-bit add of (hi, lo) into (*h, *l) with 64-bit atomics
__device__ __forceinline__ void add128(unsigned long long* h, unsigned long long* l, unsigned long long hi,
                                       unsigned long long lo) {
    const unsigned long long old = atomicAdd(l, lo);
    hi += old + lo < old ? 1ull : 0ull;
    if (hi) atomicAdd(h, hi);
}

// pass 2: the exact fixed-point sums and the shell populations
__global__ void shell_sums_kernel(const float2* __restrict__ S, int nx, int ny, int nz, int tc, int dim, double scale,
                                  int nshell, const unsigned int* __restrict__ gkey, unsigned long long* __restrict__ ghi,
                                  unsigned long long* __restrict__ glo, unsigned long long* __restrict__ gcnt) {
    extern __shared__ unsigned long long lacc[];
    unsigned long long* lhi = lacc;
    unsigned long long* llo = lacc + nshell;
    unsigned int* lcnt = reinterpret_cast<unsigned int*>(lacc + 2 * nshell);
    unsigned int* lkey = lcnt + nshell;
    for (int i = threadIdx.x; i < nshell; i += blockDim.x) {
        lhi[i] = 0ull;
        llo[i] = 0ull;
        lcnt[i] = 0u;
        lkey[i] = gkey[i];
    }
    __syncthreads();
    const int64_t total = shell_total(nx, ny, nz, dim);
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
         e += static_cast<int64_t>(gridDim.x) * blockDim.x)
        shell_terms(S, e, nx, ny, nz, tc, dim, nshell, scale, [&](int j, double t, unsigned int w) {
            atomicAdd(&lcnt[j], w);
            const int E = static_cast<int>(lkey[j] >> 1);
            if (E == 0x7ff || t == 0.0) return;  // a non-finite shell is settled by its key
            add128(&lhi[j], &llo[j], 0ull, __double2ull_rn(ldexp(t, 1084 - E)));
        });
    __syncthreads();
    for (int i = threadIdx.x; i < nshell; i += blockDim.x) {
        if (lcnt[i]) {
            add128(&ghi[i], &glo[i], lhi[i], llo[i]);
            atomicAdd(&gcnt[i], static_cast<unsigned long long>(lcnt[i]));
        }
    }
}

// pass 3: shell means S_j = sum_j / count_j, written over hi[j] as doubles
__global__ void shell_means_kernel(int nshell, const unsigned int* __restrict__ gkey,
                                   unsigned long long* __restrict__ ghi, const unsigned long long* __restrict__ glo,
                                   const unsigned long long* __restrict__ gcnt) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nshell) return;
    const unsigned int key = gkey[j];
    const int E = static_cast<int>(key >> 1);
    double v;
    if (E == 0x7ff) {
        v = (key & 1u) ? __longlong_as_double(0x7ff8000000000000ll) : __longlong_as_double(0x7ff0000000000000ll);
    } else {
        const double m = static_cast<double>(ghi[j]) * 18446744073709551616.0 + static_cast<double>(glo[j]);
        v = ldexp(m, E - 1084);
    }
    const unsigned long long n = gcnt[j];
    ghi[j] = static_cast<unsigned long long>(__double_as_longlong(n ? v / static_cast<double>(n) : 0.0));
}

// ------------------------------------------- 1D lines of mixed-radix length
// Lines whose length N = 2^a 3^b 5^c (a >= 1) is not a power of two.  One
// block per lattice keeps the spectra in LDS and transforms them with
// self-sorting (Stockham) passes of radices up to 16 (Van Loan, Sec. 1.7):
// a pass of radix r over the current length n = m r and s interleaved
// transforms maps x to
//   y[q + s (r p + j)] = w_n^(j p) sum_l x[q + s (p + l m)] w_r^(j l),
// p < m, q < s, j < r, w_n = exp(-+2 pi i / n), and the next pass takes n = m,
// s = s r, until the result stands in natural order.  The step is the one of
// the power-of-two 1D kernel, mode by mode over the whole line.

// floor(x / d) for 0 <= x < 2^21 and d >= 1, without an integer division:
// (x + 1/2)/d lies at least 1/(2d) from an integer, and rounding 1/d and the
// product moves it by less than 2^-22 (x + 1/2)/d, below 1/(2d) for such x,
// so truncating the FP32 product gives the exact quotient
struct FastDiv {
    int d;
    float rd;
    __device__ __forceinline__ explicit FastDiv(int dv) : d(dv), rd(1.0f / static_cast<float>(dv)) {}
    __device__ __forceinline__ FastDiv(int dv, float rdv) : d(dv), rd(rdv) {}
    __device__ __forceinline__ int quo(int x) const {
        return static_cast<int>((static_cast<float>(x) + 0.5f) * rd);
    }
};

// One self-sorting pass of radix R over nl lines of N values (line l at
// x + l N), sign SG = -1 (forward) or +1 (inverse): the radix-R transforms of
// the current length n = m R, then the twiddles w_n^(j p).  n s = N at every
// pass, so j p s < N indexes the table directly (the last pass, m = 1, has
// none).  Lines hold at most 2^21 values in all (they sit in LDS).
template <int R, int SG>
__device__ __forceinline__ void mr_pass(const float2* __restrict__ x, float2* __restrict__ y,
                                        const float2* __restrict__ tw, int N, int m, int s, int nl, float rper,
                                        float rs) {
    const int per = m * s;
    const FastDiv fper(per, rper), fs(s, rs);
    for (int idx = threadIdx.x; idx < nl * per; idx += blockDim.x) {
        const int line = nl == 1 ? 0 : fper.quo(idx), rem = idx - line * per;
        const int p = fs.quo(rem), q = rem - p * s;
        const float2* xl = x + line * N + rem;  // q + s p
        float2* yl = y + line * N + q + s * R * p;
        float2 a[R];
#pragma unroll
        for (int l = 0; l < R; ++l) a[l] = xl[l * per];
        DFT<R, SG>::run(a);
        if (m > 1) {
            const int ps = p * s;
#pragma unroll
            for (int j = 1; j < R; ++j) {
                float2 w = tw[j * ps];  // exp(-2 pi i j p s / N) = w_n^(j p)
                if (SG > 0) w.y = -w.y;
                a[j] = cmul(a[j], w);
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j) yl[j * s] = a[j];
    }
}

// Transform of nl lines of N values in x (LDS; line l at x + l N) with sign
// SG = -1 (forward) or +1 (inverse, unnormalised); y is LDS scratch of the
// same size.  Returns the buffer holding the result.  Every thread of the
// block calls it; it ends with a barrier.
//
// Each pass is a trip through LDS that every wave of the block waits for, so
// the passes are few: radices up to 16 in registers (MrPlan), their index
// arithmetic is kept off divisions, and the block has a thread for four
// elements.  960^2 Model B, a step: 56 us with passes of radix 4, 3, 5 on full
// spectra; 37 with half spectra and paired rows; 35 with the loads ahead of
// the transforms; 30 with passes of 10, 12 and 8.  Now 21 us a column launch
// (mostly strided access to the full state, 8 or 16 bytes of a line) and 11 us
// a row launch.
template <int SG>
__device__ __forceinline__ float2* mr_transform(float2* x, float2* y, const float2* __restrict__ tw, const MrPlan& mr,
                                                int nl = 1) {
    const int N = mr.n;
    int n = N, s = 1;
    for (int st = 0; st < mr.nst; ++st) {
        const int r = mr.radix[st];
        const float rper = mr.rper[st], rs = mr.rs[st];
        const int m = FastDiv(r, 1.0f / static_cast<float>(r)).quo(n);
        switch (r) {
            case 2: mr_pass<2, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 3: mr_pass<3, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 4: mr_pass<4, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 5: mr_pass<5, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 6: mr_pass<6, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 8: mr_pass<8, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 9: mr_pass<9, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 10: mr_pass<10, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 12: mr_pass<12, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            case 15: mr_pass<15, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
            default: mr_pass<16, SG>(x, y, tw, N, m, s, nl, rper, rs); break;
        }
        __syncthreads();
        float2* t = x;
        x = y;
        y = t;
        n = m;
        s *= r;
    }
    return x;
}

template <int NF, bool GEN, int MODE>
__global__ void __launch_bounds__(1024)
    line1d_mr_kernel(const DevPlan* __restrict__ plan, Bufs bufs, uint64_t* __restrict__ step_ctr,
                     uint32_t* __restrict__ flag, int nsteps, int advance, const float2* __restrict__ tw_g, MrPlan mr) {
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    const int N = mr.n;
    const int t = threadIdx.x, T = blockDim.x;
    float2* const tw = smem;         // exp(-2 pi i k / N)
    float2* const A = smem + N;      // transform buffers
    float2* const B = smem + 2 * N;
    float2* const S = smem + 3 * N;  // states [NF][N]
    float2* const acc = S + NF * N;  // explicit contributions [NF][N]
    float* const u = reinterpret_cast<float*>(acc + NF * N);  // de-aliased factors [ng][N]
    for (int i = t; i < N; i += T) tw[i] = tw_g[i];
    auto kq = [&](int k) { return mode_q(p, k < (N >> 1) ? k : k - N, 0, 0); };

    if constexpr (MODE == MODE_FWD_STORE) {
        for (int i = t; i < N; i += T) A[i] = make_float2(bufs.real_in[i], 0.f);
        __syncthreads();
        const float2* r = mr_transform<-1>(A, B, tw, mr);
        for (int k = t; k < N; k += T) gstore(bufs.S[bufs.sel] + k, r[k]);
        return;
    }
    if constexpr (MODE == MODE_INV_OUT) {
        for (int k = t; k < N; k += T) A[k] = gload(bufs.S[bufs.sel] + k);
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, mr);
        for (int i = t; i < N; i += T) bufs.real_out[i] = r[i].x * p.inv_n;
        return;
    }

    const int nf = p.nf;
    for (int f = 0; f < nf; ++f)
        for (int k = t; k < N; k += T) S[f * N + k] = gload(bufs.S[f] + k);
    __syncthreads();
    // Fourier value of source src (a dynamic field, or an intermediate
    // psi = sum_j op_j phi_j / (1 - L_psi)) at mode k of the current state
    auto source = [&](int src, int k, const ModeQ& q) -> float2 {
        if constexpr (GEN) {
            if (src >= PSS_MAXF) {
                const DevInterm& I = p.interm[src - PSS_MAXF];
                float2 v = make_float2(0.f, 0.f);
                for (int j = 0; j < I.nsrc; ++j) v = cadd(v, cmul(eval_op<true>(I.op[j], q), S[I.src[j] * N + k]));
                return cmul(v, cinv_implicit(1.f, eval_op<true>(I.den, q)));
            }
        }
        return S[src * N + k];
    };

    if constexpr (MODE == MODE_INTERM_OUT) {
        for (int k = t; k < N; k += T) A[k] = source(PSS_MAXF + bufs.sel, k, kq(k));
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, mr);
        for (int i = t; i < N; i += T) bufs.real_out[i] = r[i].x * p.inv_n;
        return;
    }

    // MODE_STEP: acc = sum_ch M_ch(q) F[products] from the current state
    auto channels = [&]() {
        for (int i = t; i < nf * N; i += T) acc[i] = make_float2(0.f, 0.f);
        if (p.nch == 0) {
            __syncthreads();
            return;
        }
        for (int g = 0; g < p.ng; ++g) {
            const DevMask& mk = p.mask[g];
            for (int k = t; k < N; k += T)
                A[k] = mask_keep(mk, k < (N >> 1) ? k : k - N, 0, 0) ? source(p.gfield[g], k, kq(k))
                                                                     : make_float2(0.f, 0.f);
            __syncthreads();
            const float2* r = mr_transform<1>(A, B, tw, mr);
            for (int i = t; i < N; i += T) u[g * N + i] = r[i].x * p.inv_n;
            __syncthreads();
        }
        for (int ch = 0; ch < p.nch; ++ch) {
            const DevChannel& C = p.ch[ch];
            for (int i = t; i < N; i += T) {
                float w = 0.f;
                for (int k = 0; k < C.nprod; ++k) {
                    const DevProd& pd = C.prod[k];
                    float a = pd.coef;
                    for (int g = 0; g < p.ng; ++g)
                        for (int e = 0; e < pd.pow[g]; ++e) a *= u[g * N + i];
                    w += a;
                }
                A[i] = make_float2(w, 0.f);
            }
            __syncthreads();
            const float2* r = mr_transform<-1>(A, B, tw, mr);
            for (int k = t; k < N; k += T) {
                const ModeQ q = kq(k);
                for (int o = 0; o < C.nout; ++o) {
                    float2& d = acc[C.target[o] * N + k];
                    d = cadd(d, cmul(eval_op<GEN>(C.op[o], q), r[k]));
                }
            }
            __syncthreads();
        }
    };

    const uint32_t step0 = static_cast<uint32_t>(gload_u64(step_ctr));
    uint32_t bad = 0;
    channels();
    for (int sn = 0; sn < nsteps; ++sn) {
        const uint32_t step = step0 + static_cast<uint32_t>(sn);
        // linear explicit terms from the step-n state, then the semi-implicit
        // update with the noise of this step (each mode by one thread)
        for (int k = t; k < N; k += T) {
            const ModeQ q = kq(k);
            for (int d = 0; d < p.nd; ++d) {
                const DevDirect& Dd = p.direct[d];
                float2& a = acc[Dd.target * N + k];
                a = cadd(a, cmul(eval_op<GEN>(Dd.op, q), source(Dd.src, k, q)));
            }
        }
        __syncthreads();  // the intermediates of the direct terms read every field's step-n state
        for (int k = t; k < N; k += T) {
            const ModeQ q = kq(k);
            const uint32_t lin = static_cast<uint32_t>(k), lneg = static_cast<uint32_t>((N - k) % N);
            for (int f = 0; f < nf; ++f) {
                float2 r = cadd(S[f * N + k], cscale(acc[f * N + k], p.dt));
                if (p.noisy[f] != 0) r = cadd(r, noise_mode<GEN>(p, f, step, lin, lneg, q));
                r = cmul(r, cinv_implicit(p.dt, eval_op<GEN>(p.implicit_op[f], q)));
                S[f * N + k] = r;
                if (!(__builtin_isfinite(r.x) && __builtin_isfinite(r.y))) bad |= 1u << f;
            }
        }
        __syncthreads();
        // boundary frames: the new state's real space takes the frame values
        // on the frame sites, then is transformed back
        for (int f = 0; f < nf; ++f) {
            if (p.nframe[f] == 0) continue;
            for (int k = t; k < N; k += T) A[k] = S[f * N + k];
            __syncthreads();
            float2* r = mr_transform<1>(A, B, tw, mr);
            float2* o = r == A ? B : A;
            for (int i = t; i < N; i += T) o[i] = make_float2(r[i].x * p.inv_n, 0.f);
            __syncthreads();
            const int2* __restrict__ fr = p.frame[f];
            for (int i = t; i < p.nframe[f]; i += T) o[fr[i].x] = make_float2(__int_as_float(fr[i].y), 0.f);
            __syncthreads();
            const float2* z = mr_transform<-1>(o, r, tw, mr);
            for (int k = t; k < N; k += T) S[f * N + k] = z[k];
            __syncthreads();
        }
        if (sn + 1 < nsteps) channels();
    }
    for (int f = 0; f < nf; ++f)
        for (int k = t; k < N; k += T) gstore(bufs.S[f] + k, S[f * N + k]);
    if (bad) atomicOr(flag, bad);
    __syncthreads();  // every thread has read the counter
    if (advance && t == 0) *step_ctr += static_cast<uint64_t>(nsteps);
}

hipError_t launch_line1d_mr(int mode, int N, int nf, int ng, const LaunchArgs& a) {
    MrPlan mr{};
    if (!mr_plan(N, &mr)) return hipErrorInvalidValue;
    const int NF = nf <= 1 ? 1 : (nf == 2 ? 2 : 4);
    const size_t lds = line1d_mr_lds_bytes(mr.n, NF, ng);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const dim3 grid(1), block(mr_block_threads(mr.n, 1));
    uint64_t* ctr = const_cast<uint64_t*>(a.step_ctr);
    const bool gen = a.general || mode == MODE_INTERM_OUT;
#define PSS_MR(NFV, G, M)                                                                                   \
    hipLaunchKernelGGL((line1d_mr_kernel<NFV, G, M>), grid, block, lds, a.stream, a.plan, a.bufs, ctr, a.flag, \
                       a.nsteps, a.advance != 0 ? 1 : 0, a.tw_x, mr)
#define PSS_MRF(M)                       \
    do {                                 \
        if (NF == 1) {                   \
            if (gen)                     \
                PSS_MR(1, true, M);      \
            else                         \
                PSS_MR(1, false, M);     \
        } else if (NF == 2) {            \
            if (gen)                     \
                PSS_MR(2, true, M);      \
            else                         \
                PSS_MR(2, false, M);     \
        } else {                         \
            if (gen)                     \
                PSS_MR(4, true, M);      \
            else                         \
                PSS_MR(4, false, M);     \
        }                                \
    } while (0)
    switch (mode) {
        case MODE_STEP: PSS_MRF(MODE_STEP); break;
        case MODE_INTERM_OUT: PSS_MRF(MODE_INTERM_OUT); break;
        case MODE_FWD_STORE: PSS_MR(1, false, MODE_FWD_STORE); break;
        case MODE_INV_OUT: PSS_MR(1, false, MODE_INV_OUT); break;
        default: return hipErrorInvalidValue;
    }
#undef PSS_MRF
#undef PSS_MR
    return hipGetLastError();
}

hipError_t line1d_mr_setup() {
    const int lds = 160 * 1024;
#define PSS_MRA(NFV, G, M)                                                                                     \
    if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&line1d_mr_kernel<NFV, G, M>),        \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds))                   \
        return e;
#define PSS_MRB(M) PSS_MRA(1, false, M) PSS_MRA(1, true, M) PSS_MRA(2, false, M) PSS_MRA(2, true, M) \
    PSS_MRA(4, false, M) PSS_MRA(4, true, M)
    PSS_MRB(MODE_STEP)
    PSS_MRB(MODE_INTERM_OUT)
    PSS_MRA(1, false, MODE_FWD_STORE)
    PSS_MRA(1, false, MODE_INV_OUT)
#undef PSS_MRB
#undef PSS_MRA
    return hipSuccess;
}

// ------------------------------- 2D and 3D lattices of mixed-radix sizes
// Every size an even 2^a 3^b 5^c, at least one not a power of two.  The state
// of a field is its full complex spectrum, mode (kx, ky, kz) at
// (kz Ny + ky) Nx + kx (natural order on every axis); real space is the real
// part of the inverse transform, as everywhere.  A step is launched as on the
// power-of-two path: the column kernel (lines along the last axis: forward
// transforms of the channels, the update, the de-aliased factors' inverse
// transforms), in 3D a y pass, the row kernel (inverse x transforms of the
// factors, the real-space products, their forward x transforms), in 3D a y
// pass back; each line in LDS and transformed with the self-sorting passes
// above.
//
// The products are real, so their transforms, and what real space takes from
// the factors, are Hermitian: the step's arrays hold kx = 0 .. Nx/2 only
// (layout in pss_kernels.h), one line transform serves the modes k and -k of
// the full state (the contribution to -k is the conjugate, the factor at k is
// the mean of phi(k) and conj phi(-k), which is what the real part keeps),
// and two real rows share one complex x transform.

// The addresses of a column block: tc neighbouring lines along the last axis,
// kx0 .. kx0 + nl - 1 of the half spectrum at one ky (3D), line c at c L in LDS
struct MrCols {
    int Nx, L, N1, NC, kx0, nl, ko;
    bool d3;
    __device__ __forceinline__ MrCols(const Geo& geo, int Lv, int blk) {
        Nx = geo.nx;
        L = Lv;
        N1 = geo.ny;
        NC = (Nx >> 1) + 1;
        d3 = geo.nz > 1;
        const int nxb = (NC + geo.tc - 1) / geo.tc;
        ko = d3 ? blk / nxb : 0;
        kx0 = (blk - ko * nxb) * geo.tc;
        nl = min(geo.tc, NC - kx0);
    }
    // element of a step array: line c, position w along it
    __device__ __forceinline__ size_t half(int c, int w) const {
        return d3 ? (static_cast<size_t>(ko >> 1) * NC + static_cast<size_t>(w) * (N1 >> 1) * NC + kx0 + c) * 2 + (ko & 1)
                  : (static_cast<size_t>(w >> 1) * NC + kx0 + c) * 2 + (w & 1);
    }
    // element of the state (and linear mode index): mode k of (c, w), and -k
    __device__ __forceinline__ size_t pos(int c, int w) const {
        return (d3 ? static_cast<size_t>(w) * N1 + ko : static_cast<size_t>(w)) * Nx + kx0 + c;
    }
    __device__ __forceinline__ size_t neg(int c, int w) const {
        const int kx = kx0 + c, wn = w ? L - w : 0;
        return (d3 ? static_cast<size_t>(wn) * N1 + (ko ? N1 - ko : 0) : static_cast<size_t>(wn)) * Nx + (kx ? Nx - kx : 0);
    }
    // -k lies in another column
    __device__ __forceinline__ bool paired(int c) const { return kx0 + c > 0 && 2 * (kx0 + c) < Nx; }
    __device__ __forceinline__ int w_signed(int w) const { return w < (L >> 1) ? w : w - L; }
    __device__ __forceinline__ ModeQ q(const Geo& geo, const float (&qs)[3], int c, int w) const {
        const int kx = kx0 + c, kxs = kx < (Nx >> 1) ? kx : kx - Nx, kos = ko < (N1 >> 1) ? ko : ko - N1;
        return d3 ? mode_q(Nx, N1, geo.nz, qs, kxs, kos, w_signed(w)) : mode_q(Nx, N1, 1, qs, kxs, w_signed(w), 0);
    }
};

// Column launch of a plan with one field, one channel, one factor and no
// other explicit terms (Model B): the state, its values at -k and the channel
// are read together at the top and stay in registers (at most U elements a
// thread), the operators are read once, and the new state goes straight into
// the factor's transform.  The general kernel below pays six memory latencies
// in a row; 96^2 is nothing but that.
template <int MODE>
__global__ void __launch_bounds__(1024)
    mr2_step1_kernel(const DevPlan* __restrict__ plan, const float2* __restrict__ Nin, float2* __restrict__ S,
                     float2* __restrict__ V, Geo geo, const uint64_t* __restrict__ step_ctr,
                     uint32_t* __restrict__ flag, int step_off, const float2* __restrict__ tw_g, MrPlan my) {
    constexpr bool STEP = MODE == MODE_STEP;
    constexpr int U = kMrPerThread;
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    float qs[3] = {p.qs[0], p.qs[1], p.qs[2]};
    float dt = p.dt, amp_pair = p.amp_pair, amp_self = p.amp_self;
    uint32_t key0 = p.key0, key1 = p.key1;
    int noisy = p.noisy[0], fid = p.fid[0];
    OpPoly imp = op_poly(p.implicit_op[0]), noi = op_poly(p.noise_op[0]), ch0 = op_poly(p.ch[0].op[0]);
    const int32_t* lim_g = p.lim[0];
    uint32_t step = 0;
    if constexpr (STEP) step = static_cast<uint32_t>(gload_u64(step_ctr)) + static_cast<uint32_t>(step_off);

    // XCD-ordered blocks: neighbouring columns share their cache lines in one L2
    const MrCols mc(geo, my.n, xcd_block(blockIdx.x, gridDim.x));
    const int L = mc.L, nl = mc.nl, n = nl * L;
    const int t = threadIdx.x, T = blockDim.x;
    float2* const tw = smem;
    float2* const A = smem + L;
    float2* const B = A + geo.tc * L;
    const FastDiv fnl(nl);  // n < 2^21: the LDS holds the lines
    // this thread's elements (line index fastest: a wave touches neighbouring
    // kx), the last one again past the end
    int cu[U], wu[U];
    float2 v[U], s[U], sn[U], twv[U];
    int lim[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min(t + u * T, n - 1);
        wu[u] = fnl.quo(i);
        cu[u] = i - wu[u] * nl;
        if constexpr (STEP) v[u] = gload(Nin + mc.half(cu[u], wu[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) twv[u] = tw_g[min(t + u * T, L - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        s[u] = gload(S + mc.pos(cu[u], wu[u]));
        sn[u] = gload(S + mc.neg(cu[u], wu[u]));
    }
    if constexpr (STEP) {
        hold(dt), hold(amp_pair), hold(amp_self), hold(key0), hold(key1), hold(noisy), hold(fid), hold(step);
        hold(imp), hold(noi), hold(ch0);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) hold(qs[i]);
    const bool kept = mc.kx0 < geo.ncol[0];  // some column holds kept modes (block-uniform)
    if (kept) {
        const int kos = min(mc.ko, mc.N1 - mc.ko);
#pragma unroll
        for (int u = 0; u < U; ++u) lim[u] = lim_g[(mc.d3 ? kos * mc.NC : 0) + mc.kx0 + cu[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (t + u * T < L) tw[t + u * T] = twv[u];
    float2* o = A;  // the factor's transform starts here
    float2* o2 = B;
    if constexpr (STEP) {
        // the noise, while the loads above are in flight
        float2 eta[U];
        float q2[U];
#pragma unroll
        for (int u = 0; u < U; ++u) q2[u] = mc.q(geo, qs, cu[u], wu[u]).q2;
        if (noisy) {
            const NoiseKey nk{key0, key1, step, fid, amp_pair, amp_self};
            float D[U];
            horner_p(noi, q2, D);
#pragma unroll
            for (int u = 0; u < U; ++u)
                eta[u] = u * T < n ? noise_value(nk, static_cast<uint32_t>(mc.pos(cu[u], wu[u])),
                                                 static_cast<uint32_t>(mc.neg(cu[u], wu[u])), D[u])
                                   : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (t + u * T < n) A[cu[u] * L + wu[u]] = v[u];
        __syncthreads();
        const float2* r = mr_transform<-1>(A, B, tw, my, nl);
        o = r == A ? B : A;
        o2 = r == A ? A : B;
        float M[U], Ai[U];
        horner_p(ch0, q2, M);
        horner_p(imp, q2, Ai);
        float fin = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t + u * T >= n) break;
            const float2 a = cscale(r[cu[u] * L + wu[u]], M[u]);
            float2 x = cadd(s[u], cscale(a, dt)), xn = cadd(sn[u], cscale(cconj(a), dt));
            if (noisy) {
                x = cadd(x, eta[u]);
                xn = cadd(xn, cconj(eta[u]));
            }
            const float inv = cinv_implicit(dt, make_float2(Ai[u], 0.f)).x;
            x = cscale(x, inv);
            xn = cscale(xn, inv);
            gstore(S + mc.pos(cu[u], wu[u]), x);
            fin = fmaf(x.x, 0.f, fmaf(x.y, 0.f, fin));
            if (mc.paired(cu[u])) {
                gstore(S + mc.neg(cu[u], wu[u]), xn);
                fin = fmaf(xn.x, 0.f, fmaf(xn.y, 0.f, fin));
            }
            s[u] = x;
            sn[u] = xn;
        }
        if (fin != 0.f) atomicOr(flag, 1u);  // a NaN or infinity in the new state
    }
    if (!kept) return;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (t + u * T >= n) break;
        float2 x = s[u];
        if (mc.paired(cu[u])) x = make_float2(0.5f * (x.x + sn[u].x), 0.5f * (x.y - sn[u].y));
        const int w = mc.w_signed(wu[u]);
        o[cu[u] * L + wu[u]] = w * w <= lim[u] ? x : make_float2(0.f, 0.f);
    }
    __syncthreads();
    const float2* r = mr_transform<1>(o, o2, tw, my, nl);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (t + u * T < n) gstore(V + mc.half(cu[u], wu[u]), r[cu[u] * L + wu[u]]);
}

template <int NF, bool GEN, int MODE>
__global__ void __launch_bounds__(1024)
    mr2_step_kernel(const DevPlan* __restrict__ plan, Bufs bufs, Geo geo, const uint64_t* __restrict__ step_ctr,
                    uint32_t* __restrict__ flag, int step_off, const float2* __restrict__ tw_g, MrPlan my) {
    constexpr bool STEP = MODE == MODE_STEP;
    constexpr int U = 4;  // loads issued together per thread
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    const MrCols mc(geo, my.n, xcd_block(blockIdx.x, gridDim.x));
    const int L = mc.L, nl = mc.nl, tc = geo.tc;
    const int t = threadIdx.x, T = blockDim.x;
    const int n = nl * L;
    float2* const tw = smem;
    float2* const A = smem + L;
    float2* const B = A + tc * L;
    float2* const S = B + tc * L;          // [NF][nl][L]
    float2* const acc = S + NF * tc * L;   // [NF][nl][L]
    const FastDiv fnl(nl), fL(L);  // n < 2^21: the LDS holds the lines
    auto hat = [&](int c, int w) { return mc.half(c, w); };
    auto sat = [&](int c, int w) { return mc.pos(c, w); };
    // copies between global memory (line index fastest, so that a wave touches
    // neighbouring kx) and LDS (line c at c L)
    auto gin = [&](const float2* __restrict__ src, auto at, float2* dst) {
        for (int i0 = t; i0 < n; i0 += U * T) {
            float2 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u * T, n - 1), w = fnl.quo(i);
                v[u] = gload(src + at(i - w * nl, w));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * T, w = fnl.quo(i);
                if (i < n) dst[(i - w * nl) * L + w] = v[u];
            }
        }
    };
    float qs[3] = {p.qs[0], p.qs[1], p.qs[2]};
    auto kq = [&](int c, int w) { return mc.q(geo, qs, c, w); };
    const int nf = p.nf, nch = p.nch;

    if (STEP && nch > 0) gin(bufs.N[0], hat, A);
    for (int f = 0; f < nf; ++f) gin(bufs.S[f], sat, S + f * n);
    for (int i = t; i < L; i += T) tw[i] = tw_g[i];
    if constexpr (STEP) {
        for (int i = t; i < nf * n; i += T) acc[i] = make_float2(0.f, 0.f);
    }
    __syncthreads();

    // Fourier value of source src at a mode whose fields are v: a dynamic
    // field's own, or an intermediate's (the operators at -k are the
    // conjugates of those at k, their coefficients being real)
    auto value = [&](int src, const float2 (&v)[NF][1], const ModeQ& q, bool neg) -> float2 {
        if constexpr (GEN) {
            if (src >= PSS_MAXF) {
                const DevInterm& I = p.interm[src - PSS_MAXF];
                auto at = [&](float2 o) { return neg ? cconj(o) : o; };
                float2 r = make_float2(0.f, 0.f);
                for (int j = 0; j < I.nsrc; ++j)
                    r = cadd(r, cmul(at(eval_op<true>(I.op[j], q)), pick(v, I.src[j], 0)));
                return cmul(r, cinv_implicit(1.f, at(eval_op<true>(I.den, q))));
            }
        }
        return pick(v, src, 0);
    };

    if constexpr (STEP) {
        const uint32_t step = static_cast<uint32_t>(gload_u64(step_ctr)) + static_cast<uint32_t>(step_off);
        // channels: forward transforms of the products, M(q) per mode
        for (int ch = 0; ch < nch; ++ch) {
            const DevChannel& C = p.ch[ch];
            if (ch > 0) {
                gin(bufs.N[ch], hat, A);
                __syncthreads();
            }
            const float2* r = mr_transform<-1>(A, B, tw, my, nl);
            for (int i = t; i < n; i += T) {
                const int c = fL.quo(i), w = i - c * L;
                const ModeQ q = kq(c, w);
                for (int o = 0; o < C.nout; ++o) {
                    float2& d = acc[C.target[o] * n + i];
                    d = cadd(d, cmul(eval_op<GEN>(C.op[o], q), r[i]));
                }
            }
            __syncthreads();
        }
        // linear explicit terms from the step-n state, then the semi-implicit
        // update with the noise, of k and (paired columns) of -k; S keeps what
        // the factors take of the new state.  Each element by one thread, the
        // line index fastest (the state's stores).
        uint32_t bad = 0;
        for (int i0 = t; i0 < n; i0 += U * T) {
            float2 sn[U][NF][1];  // the states at -k
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u * T, n - 1), w = fnl.quo(i);
                const size_t e = mc.neg(i - w * nl, w);
#pragma unroll
                for (int f = 0; f < NF; ++f) sn[u][f][0] = f < nf ? gload(bufs.S[f] + e) : make_float2(0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * T;
                if (i >= n) break;
                const int w = fnl.quo(i), c = i - w * nl, e = c * L + w;
                const bool pr = mc.paired(c);
                const ModeQ q = kq(c, w);
                const uint32_t lin = static_cast<uint32_t>(sat(c, w)), lneg = static_cast<uint32_t>(mc.neg(c, w));
                float2 sv[NF][1], a[NF][1], an[NF][1];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    sv[f][0] = f < nf ? S[f * n + e] : make_float2(0.f, 0.f);
                    a[f][0] = f < nf ? acc[f * n + e] : make_float2(0.f, 0.f);
                    an[f][0] = cconj(a[f][0]);
                }
                for (int d = 0; d < p.nd; ++d) {
                    const DevDirect& Dd = p.direct[d];
                    const float2 op = eval_op<GEN>(Dd.op, q);
                    add_to(a, Dd.target, 0, cmul(op, value(Dd.src, sv, q, false)));
                    add_to(an, Dd.target, 0, cmul(cconj(op), value(Dd.src, sn[u], q, true)));
                }
                static_for<NF>([&](auto FF) {
                    constexpr int f = decltype(FF)::value;
                    if (f >= nf) return;
                    float2 r = cadd(sv[f][0], cscale(a[f][0], p.dt)), rn = cadd(sn[u][f][0], cscale(an[f][0], p.dt));
                    if (p.noisy[f] != 0) {
                        const float2 eta = noise_mode<GEN>(p, f, step, lin, lneg, q);
                        r = cadd(r, eta);
                        rn = cadd(rn, cconj(eta));
                    }
                    const float2 inv = cinv_implicit(p.dt, eval_op<GEN>(p.implicit_op[f], q));
                    r = cmul(r, inv);
                    gstore(bufs.S[f] + lin, r);
                    bool fin = __builtin_isfinite(r.x) && __builtin_isfinite(r.y);
                    if (pr) {
                        rn = cmul(rn, cconj(inv));
                        gstore(bufs.S[f] + lneg, rn);
                        fin = fin && __builtin_isfinite(rn.x) && __builtin_isfinite(rn.y);
                        r = make_float2(0.5f * (r.x + rn.x), 0.5f * (r.y - rn.y));
                    }
                    if (!fin) bad |= 1u << f;
                    S[f * n + e] = r;
                });
            }
        }
        if (bad) atomicOr(flag, bad);
        __syncthreads();
    } else {
        // S: what the factors take of the state
        for (int i = t; i < n; i += T) {
            const int w = fnl.quo(i), c = i - w * nl, e = c * L + w;
            if (!mc.paired(c)) continue;
            for (int f = 0; f < nf; ++f) {
                const float2 a = S[f * n + e], b = gload(bufs.S[f] + mc.neg(c, w));
                S[f * n + e] = make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
            }
        }
        __syncthreads();
    }

    // inverse transforms of the de-aliased factors
    for (int g = 0; g < p.ng; ++g) {
        if (mc.kx0 >= geo.ncol[g]) continue;  // every column masked: never read (block-uniform)
        // the largest kept w^2 of each line
        const int32_t* lim = p.lim[g] + (mc.d3 ? min(mc.ko, mc.N1 - mc.ko) * mc.NC : 0) + mc.kx0;
        for (int i = t; i < n; i += T) {
            const int c = fL.quo(i), w = i - c * L;
            float2 v = make_float2(0.f, 0.f);
            if (mc.w_signed(w) * mc.w_signed(w) <= lim[c]) {
                float2 sv[NF][1];
#pragma unroll
                for (int f = 0; f < NF; ++f) sv[f][0] = f < nf ? S[f * n + i] : make_float2(0.f, 0.f);
                v = value(p.gfield[g], sv, kq(c, w), false);
            }
            A[i] = v;
        }
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, my, nl);
        for (int i = t; i < n; i += T) {
            const int w = fnl.quo(i), c = i - w * nl;
            gstore(bufs.V[g] + hat(c, w), r[c * L + w]);
        }
        if (g + 1 < p.ng) __syncthreads();
    }
}

// Row launch of a step: ROWS = 2 rows per block (one where two do not fit the
// LDS), as one complex line Z = X1 + i X2
template <int ROWS, bool ONE>
__global__ void __launch_bounds__(1024)
    mr2_prod_kernel(const DevPlan* __restrict__ plan, Bufs bufs, Geo geo, const float2* __restrict__ tw_g, MrPlan mx,
                    int64_t advance, uint64_t* __restrict__ step_ctr) {
    constexpr int U = 2;
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    const int Nx = mx.n, NH = Nx >> 1, NC = NH + 1;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    // the block's pair of rows and, of one row, which it is
    const size_t pair = static_cast<size_t>(ROWS == 2 ? blk : blk >> 1) * NC * 2;
    const int odd = ROWS == 2 ? 0 : blk & 1;
    const int t = threadIdx.x, T = blockDim.x;
    float2* const tw = smem;
    float2* const A = smem + Nx;
    float2* const B = smem + 2 * Nx;
    float* const u = reinterpret_cast<float*>(smem + 3 * Nx);  // [ng][Nx][ROWS]
    int ng = p.ng, nch = p.nch, np0 = p.ch[0].nprod;
    float inv_n = p.inv_n, c0 = p.ch[0].prod[0].coef;
    int pw0 = p.ch[0].prod[0].pow[0];
    // Z[c] and Z[Nx - c] from column c of both rows (columns from ncol on are
    // zero); of columns 0 and Nx/2 real space takes the real parts
    auto gather = [&](const float2* __restrict__ src, int ncol) {
        for (int c0 = t; c0 < NC; c0 += U * T) {
            float2 x[U], y[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int c = min(c0 + k * T, NC - 1), cl = c < ncol ? c : 0;
                const float2* e = src + pair + static_cast<size_t>(cl) * 2;
                if constexpr (ROWS == 2) {
                    gload_pair(e, x[k], y[k]);
                } else {
                    x[k] = gload(e + odd);
                    y[k] = make_float2(0.f, 0.f);
                }
                if (c >= ncol) x[k] = y[k] = make_float2(0.f, 0.f);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int c = c0 + k * T;
                if (c >= NC) break;
                if (c == 0 || c == NH) {
                    A[c] = make_float2(x[k].x, y[k].x);
                } else {
                    A[c] = make_float2(x[k].x - y[k].y, x[k].y + y[k].x);
                    A[Nx - c] = make_float2(x[k].x + y[k].y, y[k].x - x[k].y);
                }
            }
        }
    };
    // unpack the rows of a transform and store their columns 0 .. Nx/2
    auto store = [&](const float2* r, float2* __restrict__ dst) {
        for (int c = t; c < NC; c += T) {
            const float2 a = r[c], b = r[c == 0 ? 0 : Nx - c];
            float2* e = dst + pair + static_cast<size_t>(c) * 2;
            const float2 x1 = make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
            if constexpr (ROWS == 2) {
                gstore_pair_sel<false>(e, x1, make_float2(0.5f * (a.y + b.y), 0.5f * (b.x - a.x)));
            } else {
                gstore(e + odd, x1);
            }
        }
    };
    gather(bufs.V[0], geo.ncol[0]);
    for (int i = t; i < Nx; i += T) tw[i] = tw_g[i];
    hold(ng), hold(nch), hold(np0), hold(inv_n), hold(c0), hold(pw0);
    if constexpr (ONE) {
        // one factor and one channel: the products go from one transform's
        // result straight into the other's input
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, mx);
        float2* const o = r == A ? B : A;
        float2* const o2 = r == A ? A : B;
        for (int x = t; x < Nx; x += T) {
            const float2 z[1] = {cscale(r[x], inv_n)};
            float2 w = make_float2(0.f, 0.f);
            for (int k = 0; k < np0; ++k) {
                const float cf = k == 0 ? c0 : p.ch[0].prod[k].coef;
                const int pw = k == 0 ? pw0 : p.ch[0].prod[k].pow[0];
                float2 a[1] = {make_float2(cf, cf)};
                times_power<0>(a, z, pw);
                w = cadd(w, a[0]);
            }
            if (ROWS == 1) w.y = 0.f;
            o[x] = w;
        }
        __syncthreads();
        store(mr_transform<-1>(o, o2, tw, mx), bufs.N[0]);
        if (advance != 0 && blk == 0 && t == 0) *step_ctr += static_cast<uint64_t>(advance);
        return;
    }
    for (int g = 0; g < ng; ++g) {
        if (g > 0) gather(bufs.V[g], geo.ncol[g]);
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, mx);
        for (int x = t; x < Nx; x += T) {
            const float2 v = r[x];
            u[(g * Nx + x) * ROWS] = v.x * inv_n;
            if constexpr (ROWS == 2) u[(g * Nx + x) * ROWS + 1] = v.y * inv_n;
        }
        __syncthreads();
    }
    for (int ch = 0; ch < nch; ++ch) {
        const DevChannel& C = p.ch[ch];
        for (int x = t; x < Nx; x += T) {
            float w[2] = {0.f, 0.f};
            for (int k = 0; k < C.nprod; ++k) {
                const DevProd& pd = C.prod[k];
                float a[2] = {pd.coef, pd.coef};
                for (int g = 0; g < ng; ++g) {
                    const int pw = pd.pow[g];
                    if (pw == 0) continue;
                    float z[ROWS];
#pragma unroll
                    for (int j = 0; j < ROWS; ++j) z[j] = u[(g * Nx + x) * ROWS + j];
                    for (int e = 0; e < pw; ++e) {
#pragma unroll
                        for (int j = 0; j < ROWS; ++j) a[j] *= z[j];
                    }
                }
#pragma unroll
                for (int j = 0; j < ROWS; ++j) w[j] += a[j];
            }
            A[x] = make_float2(w[0], w[1]);
        }
        __syncthreads();
        const float2* r = mr_transform<-1>(A, B, tw, mx);
        store(r, bufs.N[ch]);
        if (ch + 1 < nch) __syncthreads();
    }
    if (advance != 0 && blk == 0 && t == 0) *step_ctr += static_cast<uint64_t>(advance);
}

// the transform modes of full spectra
template <int NF, bool GEN, int MODE>
__global__ void __launch_bounds__(1024)
    mr2_col_kernel(const DevPlan* __restrict__ plan, Bufs bufs, const float2* __restrict__ tw_g, MrPlan my, int tc) {
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    // tc neighbouring lines along the last axis: y in 2D (block = kx0 ..
    // kx0 + tc - 1), z in 3D (the same kx range at one ky); "ky" below is the
    // index along a line.  LDS holds line c of an array at c L.
    const int Nx = p.n[0], L = my.n, N1 = p.n[1];
    const bool d3 = p.n[2] > 1;
    const int nxb = Nx / tc;
    // XCD-ordered blocks: each XCD's L2 takes a contiguous range of columns,
    // so the cache lines that neighbouring column blocks share are fetched
    // into one L2, not into all eight
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int kx0 = (blk % nxb) * tc;
    const int ko = d3 ? blk / nxb : 0;  // ky of 3D lines
    const int kos = ko < (N1 >> 1) ? ko : ko - N1;
    const size_t base = d3 ? static_cast<size_t>(ko) * Nx + kx0 : static_cast<size_t>(kx0);
    const size_t su = d3 ? static_cast<size_t>(Nx) * N1 : static_cast<size_t>(Nx);
    const int t = threadIdx.x, T = blockDim.x;
    const int n = tc * L;  // elements of one array in LDS
    float2* const tw = smem;
    float2* const A = smem + L;
    float2* const B = A + n;
    float2* const S = B + n;          // [NF][tc][L]
    for (int i = t; i < L; i += T) tw[i] = tw_g[i];
    const FastDiv ftc(tc), fL(L);  // n < 2^21: the LDS holds the lines
    // global element of line c at position w; loads and stores run with the
    // line index fastest, so a wave touches neighbouring kx
    auto at = [&](int c, int w) { return base + c + static_cast<size_t>(w) * su; };
    auto gin = [&](const float2* __restrict__ src, float2* dst) {
        for (int i = t; i < n; i += T) {
            const int w = ftc.quo(i), c = i - w * tc;
            dst[c * L + w] = gload(src + at(c, w));
        }
    };
    auto gout = [&](const float2* src, float2* __restrict__ dst) {
        for (int i = t; i < n; i += T) {
            const int w = ftc.quo(i), c = i - w * tc;
            gstore(dst + at(c, w), src[c * L + w]);
        }
    };
    // line and position of LDS element i
    auto lw = [&](int i, int& c, int& w) {
        c = fL.quo(i);
        w = i - c * L;
    };
    auto ws = [&](int w) { return w < (L >> 1) ? w : w - L; };
    auto kxs = [&](int c) { const int kx = kx0 + c; return kx < (Nx >> 1) ? kx : kx - Nx; };
    auto kq = [&](int c, int w) { return d3 ? mode_q(p, kxs(c), kos, ws(w)) : mode_q(p, kxs(c), ws(w), 0); };

    if constexpr (MODE == MODE_FWD_STORE) {
        gin(bufs.in, A);
        __syncthreads();
        const float2* r = mr_transform<-1>(A, B, tw, my, tc);
        gout(r, bufs.S[bufs.sel]);
        return;
    }
    if constexpr (MODE == MODE_INV_OUT) {
        gin(bufs.S[bufs.sel], A);
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, my, tc);
        gout(r, bufs.out);
        return;
    }

    const int nf = p.nf;
    for (int f = 0; f < nf; ++f) gin(bufs.S[f], S + f * n);
    __syncthreads();
    // Fourier value of source src at LDS element i (line i / L, position i % L)
    auto source = [&](int src, int i, const ModeQ& q) -> float2 {
        if constexpr (GEN) {
            if (src >= PSS_MAXF) {
                const DevInterm& I = p.interm[src - PSS_MAXF];
                float2 v = make_float2(0.f, 0.f);
                for (int j = 0; j < I.nsrc; ++j) v = cadd(v, cmul(eval_op<true>(I.op[j], q), S[I.src[j] * n + i]));
                return cmul(v, cinv_implicit(1.f, eval_op<true>(I.den, q)));
            }
        }
        return S[src * n + i];
    };

    // MODE_INTERM_OUT
    for (int i = t; i < n; i += T) {
        int c, w;
        lw(i, c, w);
        A[i] = source(PSS_MAXF + bufs.sel, i, kq(c, w));
    }
    __syncthreads();
    const float2* r = mr_transform<1>(A, B, tw, my, tc);
    gout(r, bufs.out);
    }

template <int MODE>
__global__ void __launch_bounds__(1024)
    mr2_row_kernel(const DevPlan* __restrict__ plan, Bufs bufs, const float2* __restrict__ tw_g, MrPlan mx) {
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    const int Nx = mx.n;
    const size_t row = static_cast<size_t>(blockIdx.x) * Nx;
    const int t = threadIdx.x, T = blockDim.x;
    float2* const tw = smem;
    float2* const A = smem + Nx;
    float2* const B = smem + 2 * Nx;
    for (int i = t; i < Nx; i += T) tw[i] = tw_g[i];

    if constexpr (MODE == MODE_R2C_IN) {
        for (int x = t; x < Nx; x += T) A[x] = make_float2(bufs.real_in[row + x], 0.f);
        __syncthreads();
        const float2* r = mr_transform<-1>(A, B, tw, mx);
        for (int k = t; k < Nx; k += T) gstore(bufs.out + row + k, r[k]);
        return;
    }
    if constexpr (MODE == MODE_C2R_OUT) {
        for (int k = t; k < Nx; k += T) A[k] = gload(bufs.in + row + k);
        __syncthreads();
        const float2* r = mr_transform<1>(A, B, tw, mx);
        for (int x = t; x < Nx; x += T) bufs.real_out[row + x] = r[x].x * p.inv_n;
        return;
    }
}

// 3D: transforms along y of the arrays of ya (in place allowed: a line is
// read whole before it is written), tc lines of neighbouring kx at one z per
// block; half spectra (only columns below ya.ncol are read later) or full ones
template <int SG, bool FULL>
__global__ void __launch_bounds__(1024)
    mr3_ypass_kernel(YArgs ya, Geo geo, const float2* __restrict__ tw_g, MrPlan my, int tc) {
    extern __shared__ float2 smem[];
    const int Nx = geo.nx, Ny = my.n, NK = FULL ? Nx : (Nx >> 1) + 1;
    const int nxb = (NK + tc - 1) / tc;
    const int blk = xcd_block(blockIdx.x, gridDim.x);  // as in the column kernel
    const int z = blk / nxb, kx0 = (blk - z * nxb) * tc;
    const int nl = min(tc, NK - kx0);
    const int t = threadIdx.x, T = blockDim.x;
    const int n = nl * Ny;
    const FastDiv fnl(nl);
    float2* const tw = smem;
    float2* const A = smem + Ny;
    float2* const B = A + tc * Ny;
    auto at = [&](int c, int y) {
        return FULL ? (static_cast<size_t>(z) * Ny + y) * Nx + kx0 + c
                    : ((static_cast<size_t>(z) * (Ny >> 1) + (y >> 1)) * NK + kx0 + c) * 2 + (y & 1);
    };
    for (int i = t; i < Ny; i += T) tw[i] = tw_g[i];
    for (int a = 0; a < ya.n; ++a) {
        if (!FULL && kx0 >= ya.ncol[a]) continue;  // block-uniform
        for (int i = t; i < n; i += T) {
            const int y = fnl.quo(i), c = i - y * nl;
            A[c * Ny + y] = gload(ya.src[a] + at(c, y));
        }
        __syncthreads();
        const float2* r = mr_transform<SG>(A, B, tw, my, nl);
        for (int i = t; i < n; i += T) {
            const int y = fnl.quo(i), c = i - y * nl;
            gstore(ya.dst[a] + at(c, y), r[c * Ny + y]);
        }
        __syncthreads();
    }
}

hipError_t launch_mr3_ypass(int sign, const YArgs& ya, bool full, const LaunchArgs& a) {
    MrPlan my{};
    if (!mr_plan(a.ny, &my) || a.dim != 3) return hipErrorInvalidValue;
    if (ya.n <= 0) return hipSuccess;
    const int tc = a.geo.py;  // neighbouring y lines per block
    if (tc < 1 || a.nx % tc != 0) return hipErrorInvalidValue;
    const size_t lds = mr3_ypass_lds_bytes(my.n, tc);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const int nk = full ? a.nx : a.nx / 2 + 1;
    const dim3 grid(((nk + tc - 1) / tc) * a.nz), block(mr_threads(tc * my.n));
#define PSS_Y3(SG, F) hipLaunchKernelGGL((mr3_ypass_kernel<SG, F>), grid, block, lds, a.stream, ya, a.geo, a.tw_y, my, tc)
    if (sign < 0) {
        if (full)
            PSS_Y3(-1, true);
        else
            PSS_Y3(-1, false);
    } else {
        if (full)
            PSS_Y3(1, true);
        else
            PSS_Y3(1, false);
    }
#undef PSS_Y3
    return hipGetLastError();
}

hipError_t launch_mr2_col(int mode, int nf, const LaunchArgs& a) {
    MrPlan my{};
    if (!mr_plan(a.dim == 3 ? a.nz : a.ny, &my)) return hipErrorInvalidValue;
    const int NF = nf <= 1 ? 1 : (nf == 2 ? 2 : 4);
    const int tc = a.geo.tc;  // neighbouring lines per block
    if (tc < 1 || a.nx % tc != 0) return hipErrorInvalidValue;
    const size_t lds = mr2_col_lds_bytes(my.n, NF, tc);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const int other = a.dim == 3 ? a.ny : 1;
    const dim3 full((a.nx / tc) * other), half(((a.nx / 2 + tc) / tc) * other), block(mr_threads(tc * my.n));
    const dim3 wide(mr_block_threads(tc * my.n, half.x));
    const bool gen = a.general;
#define PSS_C2(NFV, G, M)                                                                                         \
    hipLaunchKernelGGL((mr2_step_kernel<NFV, G, M>), half, wide, lds, a.stream, a.plan, a.bufs, a.geo, a.step_ctr, \
                       a.flag, a.step_off, a.tw_u, my)
    // one element per thread and load slot: the lines of the block fit
    const bool one = a.simple && tc * my.n <= kMrPerThread * static_cast<int>(block.x);
#define PSS_C1(M)                                                                                              \
    hipLaunchKernelGGL((mr2_step1_kernel<M>), half, block, lds1, a.stream, a.plan, a.bufs.N[0], a.bufs.S[0],   \
                       a.bufs.V[0], a.geo, a.step_ctr, a.flag, a.step_off, a.tw_u, my)
    const size_t lds1 = mr3_ypass_lds_bytes(my.n, tc);  // twiddles and two buffers
#define PSS_C2F(M)                       \
    do {                                 \
        if (one) {                       \
            PSS_C1(M);                   \
        } else if (NF == 1) {            \
            if (gen)                     \
                PSS_C2(1, true, M);      \
            else                         \
                PSS_C2(1, false, M);     \
        } else if (NF == 2) {            \
            if (gen)                     \
                PSS_C2(2, true, M);      \
            else                         \
                PSS_C2(2, false, M);     \
        } else {                         \
            if (gen)                     \
                PSS_C2(4, true, M);      \
            else                         \
                PSS_C2(4, false, M);     \
        }                                \
    } while (0)
#define PSS_CT(NFV, G, M) \
    hipLaunchKernelGGL((mr2_col_kernel<NFV, G, M>), full, block, lds, a.stream, a.plan, a.bufs, a.tw_u, my, tc)
    switch (mode) {
        case MODE_STEP: PSS_C2F(MODE_STEP); break;
        case MODE_PROLOGUE: PSS_C2F(MODE_PROLOGUE); break;
        case MODE_INTERM_OUT:
            if (NF == 1)
                PSS_CT(1, true, MODE_INTERM_OUT);
            else if (NF == 2)
                PSS_CT(2, true, MODE_INTERM_OUT);
            else
                PSS_CT(4, true, MODE_INTERM_OUT);
            break;
        case MODE_FWD_STORE: PSS_CT(1, false, MODE_FWD_STORE); break;
        case MODE_INV_OUT: PSS_CT(1, false, MODE_INV_OUT); break;
        default: return hipErrorInvalidValue;
    }
#undef PSS_CT
#undef PSS_C1
#undef PSS_C2F
#undef PSS_C2
    return hipGetLastError();
}

hipError_t launch_mr2_row(int mode, const LaunchArgs& a) {
    MrPlan mx{};
    if (!mr_plan(a.nx, &mx)) return hipErrorInvalidValue;
    const int rows = a.ny * (a.dim == 3 ? a.nz : 1);
    const int per = mode == MODE_STEP ? mr2_rows(mx.n, a.ng) : 1;
    const size_t lds = mr2_row_lds_bytes(mx.n, mode == MODE_STEP ? a.ng : 1, per);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const dim3 grid(rows / per);
    const dim3 block(mode == MODE_STEP && !a.simple ? mr_block_threads(mx.n, grid.x) : mr_threads(mx.n));
    uint64_t* ctr = const_cast<uint64_t*>(a.step_ctr);
    switch (mode) {
        case MODE_STEP:
#define PSS_PR(R, ONE)                                                                                         \
    hipLaunchKernelGGL((mr2_prod_kernel<R, ONE>), grid, block, lds, a.stream, a.plan, a.bufs, a.geo, a.tw_x, mx, \
                       a.advance, ctr)
            if (per == 2) {
                if (a.simple)
                    PSS_PR(2, true);
                else
                    PSS_PR(2, false);
            } else {
                if (a.simple)
                    PSS_PR(1, true);
                else
                    PSS_PR(1, false);
            }
#undef PSS_PR
            break;
        case MODE_R2C_IN:
            hipLaunchKernelGGL(mr2_row_kernel<MODE_R2C_IN>, grid, block, lds, a.stream, a.plan, a.bufs, a.tw_x, mx);
            break;
        case MODE_C2R_OUT:
            hipLaunchKernelGGL(mr2_row_kernel<MODE_C2R_OUT>, grid, block, lds, a.stream, a.plan, a.bufs, a.tw_x, mx);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t mr2_setup() {
    const int lds = 160 * 1024;
#define PSS_LDS(...)                                                                     \
    if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&(__VA_ARGS__)), \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds)) \
        return e;
#define PSS_C2B(M)                                                                                     \
    PSS_LDS(mr2_step_kernel<1, false, M>) PSS_LDS(mr2_step_kernel<1, true, M>)                         \
    PSS_LDS(mr2_step_kernel<2, false, M>) PSS_LDS(mr2_step_kernel<2, true, M>)                         \
    PSS_LDS(mr2_step_kernel<4, false, M>) PSS_LDS(mr2_step_kernel<4, true, M>)
    PSS_C2B(MODE_STEP)
    PSS_C2B(MODE_PROLOGUE)
#undef PSS_C2B
    PSS_LDS(mr2_col_kernel<1, true, MODE_INTERM_OUT>)
    PSS_LDS(mr2_col_kernel<2, true, MODE_INTERM_OUT>)
    PSS_LDS(mr2_col_kernel<4, true, MODE_INTERM_OUT>)
    PSS_LDS(mr2_col_kernel<1, false, MODE_FWD_STORE>)
    PSS_LDS(mr2_col_kernel<1, false, MODE_INV_OUT>)
    PSS_LDS(mr2_prod_kernel<1, false>)
    PSS_LDS(mr2_prod_kernel<2, false>)
    PSS_LDS(mr2_prod_kernel<1, true>)
    PSS_LDS(mr2_prod_kernel<2, true>)
    PSS_LDS(mr2_step1_kernel<MODE_STEP>)
    PSS_LDS(mr2_step1_kernel<MODE_PROLOGUE>)
    PSS_LDS(mr2_row_kernel<MODE_R2C_IN>)
    PSS_LDS(mr2_row_kernel<MODE_C2R_OUT>)
    PSS_LDS(mr3_ypass_kernel<-1, false>)
    PSS_LDS(mr3_ypass_kernel<-1, true>)
    PSS_LDS(mr3_ypass_kernel<1, false>)
    PSS_LDS(mr3_ypass_kernel<1, true>)
#undef PSS_LDS
    return hipSuccess;
}
#endif  // PSS_COMMON

// ------------------------------------------------------- launch dispatch
// -------------------------------------------------------------- 1D lattices
// One block holds the whole line of N sites: T = N/4 threads, 4 modes each.
// A field's state is its full complex spectrum (Hermitian up to rounding) in
// natural mode order; thread t keeps modes k = D(t) + m T, the order in which
// the forward transform leaves them and the inverse transform takes them, so
// a step needs no reordering.  Real space is the real part of the inverse
// transform (as for every dimension).  A launch first forms the explicit
// contributions of its first step from the state, then takes its steps in
// registers, following the per-step list after eq:timeupdate: intermediate
// and de-aliased factors from the state, inverse transforms, products,
// forward transforms, noise, semi-implicit update.
template <int N, int NF, bool GEN, int MODE>
__global__ void __launch_bounds__(N / 4 < 64 ? 64 : N / 4)
    line1d_kernel(const DevPlan* __restrict__ plan, Bufs bufs, uint64_t* __restrict__ step_ctr,
                  uint32_t* __restrict__ flag, int nsteps, int advance, const float2* __restrict__ tw_g) {
    constexpr int P = 4;
    using FFT = LineFFT<N, P>;
    constexpr int T = FFT::T;
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    const int t = threadIdx.x;
    LdsLine ld = FFT::lds_line(smem);
    float2* const twl = smem + FFT::kLds;
    float* const xst = reinterpret_cast<float*>(twl + N);  // real-space staging of the frames
    for (int i = t; i < N; i += T) twl[i] = tw_g[i];
    __syncthreads();
    const float2* tw = twl;
    const int dr = FFT::drev(t);
    // the modes of this thread: index k = dr + m T, signed kx, q, linear indices
    ModeQ q[P];
    float q2[P];
    uint32_t lin[P], lneg[P];
#pragma unroll
    for (int m = 0; m < P; ++m) {
        const int k = dr + m * T;
        q[m] = mode_q(p, k < (N >> 1) ? k : k - N, 0, 0);
        q2[m] = q[m].q2;
        lin[m] = static_cast<uint32_t>(k);
        lneg[m] = static_cast<uint32_t>((N - k) & (N - 1));
    }

    if constexpr (MODE == MODE_FWD_STORE) {
        float2 v[P];
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = make_float2(bufs.real_in[t + m * T], 0.f);
        FFT::template dif<-1>(v, ld, t, tw);
#pragma unroll
        for (int m = 0; m < P; ++m) gstore(bufs.S[bufs.sel] + dr + m * T, v[m]);
        return;
    }
    if constexpr (MODE == MODE_INV_OUT) {
        float2 v[P];
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = gload(bufs.S[bufs.sel] + dr + m * T);
        FFT::template dit<1>(v, ld, t, tw);
#pragma unroll
        for (int m = 0; m < P; ++m) bufs.real_out[t + m * T] = v[m].x * p.inv_n;
        return;
    }

    float2 s[NF][P];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int m = 0; m < P; ++m) s[f][m] = f < p.nf ? gload(bufs.S[f] + dr + m * T) : make_float2(0.f, 0.f);

    // the Fourier values of source `src` (a dynamic field, or an intermediate
    // psi = sum_k op_k phi_k / (1 - L_psi)) at this thread's modes
    auto source = [&](int src, float2 (&v)[P]) {
        if constexpr (GEN) {
            if (src >= PSS_MAXF) {
                const DevInterm& I = p.interm[src - PSS_MAXF];
#pragma unroll
                for (int m = 0; m < P; ++m) v[m] = make_float2(0.f, 0.f);
                for (int k = 0; k < I.nsrc; ++k) {
                    const int sk = I.src[k];
#pragma unroll
                    for (int m = 0; m < P; ++m) v[m] = cadd(v[m], cmul(eval_op<true>(I.op[k], q[m]), pick(s, sk, m)));
                }
#pragma unroll
                for (int m = 0; m < P; ++m) v[m] = cmul(v[m], cinv_implicit(1.f, eval_op<true>(I.den, q[m])));
                return;
            }
        }
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = pick(s, src, m);
    };

    if constexpr (MODE == MODE_INTERM_OUT) {
        float2 v[P];
        source(PSS_MAXF + bufs.sel, v);
        FFT::template dit<1>(v, ld, t, tw);
#pragma unroll
        for (int m = 0; m < P; ++m) bufs.real_out[t + m * T] = v[m].x * p.inv_n;
        return;
    }

    // MODE_STEP.  acc: the explicit contributions sum_ch M_ch(q) F[products]
    float2 acc[NF][P];
    auto channels = [&]() {
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int m = 0; m < P; ++m) acc[f][m] = make_float2(0.f, 0.f);
        if (p.nch == 0) return;
        // real-space values of the de-aliased factors at x = t + m T
        float u[PSS_MAXG][P];
#pragma unroll
        for (int g = 0; g < PSS_MAXG; ++g) {
            if (g >= p.ng) break;
            const DevMask& mk = p.mask[g];
            float2 v[P];
            source(p.gfield[g], v);
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const int k = dr + m * T;
                if (!mask_keep(mk, k < (N >> 1) ? k : k - N, 0, 0)) v[m] = make_float2(0.f, 0.f);
            }
            FFT::template dit<1>(v, ld, t, tw);
#pragma unroll
            for (int m = 0; m < P; ++m) u[g][m] = v[m].x * p.inv_n;
        }
        for (int ch = 0; ch < p.nch; ++ch) {
            const DevChannel& C = p.ch[ch];
            float2 w[P];
#pragma unroll
            for (int m = 0; m < P; ++m) w[m] = make_float2(0.f, 0.f);
            for (int k = 0; k < C.nprod; ++k) {
                const DevProd& pd = C.prod[k];
                uint64_t pw;
                __builtin_memcpy(&pw, pd.pow, sizeof(pw));
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    float a = pd.coef;
#pragma unroll
                    for (int g = 0; g < PSS_MAXG; ++g) {
                        if (g >= p.ng) break;
                        const int pg = static_cast<int>((pw >> (8 * g)) & 0xffull);
                        for (int e = 0; e < pg; ++e) a *= u[g][m];
                    }
                    w[m].x += a;
                }
            }
            FFT::template dif<-1>(w, ld, t, tw);
            for (int o = 0; o < C.nout; ++o)
#pragma unroll
                for (int m = 0; m < P; ++m) add_to(acc, C.target[o], m, cmul(eval_op<GEN>(C.op[o], q[m]), w[m]));
        }
    };

    const uint32_t step0 = static_cast<uint32_t>(gload_u64(step_ctr));
    uint32_t bad = 0;
    channels();
    for (int sn = 0; sn < nsteps; ++sn) {
        const uint32_t step = step0 + static_cast<uint32_t>(sn);
        // linear explicit terms from the step-n state
        for (int d = 0; d < p.nd; ++d) {
            const DevDirect& Dd = p.direct[d];
            float2 src[P];
            source(Dd.src, src);
#pragma unroll
            for (int m = 0; m < P; ++m) add_to(acc, Dd.target, m, cmul(eval_op<GEN>(Dd.op, q[m]), src[m]));
        }
        // semi-implicit update with the noise of this step
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (f >= p.nf) continue;
            const bool noisy = p.noisy[f] != 0;
#pragma unroll
            for (int m = 0; m < P; ++m) {
                float2 r = cadd(s[f][m], cscale(acc[f][m], p.dt));
                if (noisy) r = cadd(r, noise_mode<GEN>(p, f, step, lin[m], lneg[m], q[m]));
                s[f][m] = cmul(r, cinv_implicit(p.dt, eval_op<GEN>(p.implicit_op[f], q[m])));
            }
        }
        // boundary frames: the new state's real space takes the frame values
        // on the frame sites (staged through LDS), then is transformed back
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (f >= p.nf || p.nframe[f] == 0) continue;
            float2 v[P];
#pragma unroll
            for (int m = 0; m < P; ++m) v[m] = s[f][m];
            FFT::template dit<1>(v, ld, t, tw);
#pragma unroll
            for (int m = 0; m < P; ++m) xst[t + m * T] = v[m].x * p.inv_n;
            __syncthreads();
            const int2* __restrict__ fr = p.frame[f];
            for (int i = t; i < p.nframe[f]; i += T) {
                const int2 e = fr[i];
                xst[e.x] = __int_as_float(e.y);
            }
            __syncthreads();
#pragma unroll
            for (int m = 0; m < P; ++m) v[m] = make_float2(xst[t + m * T], 0.f);
            __syncthreads();  // the staging line is free again
            FFT::template dif<-1>(v, ld, t, tw);
#pragma unroll
            for (int m = 0; m < P; ++m) s[f][m] = v[m];
        }
#pragma unroll
        for (int f = 0; f < NF; ++f)
            if (f < p.nf)
#pragma unroll
                for (int m = 0; m < P; ++m)
                    if (!(__builtin_isfinite(s[f][m].x) && __builtin_isfinite(s[f][m].y))) bad |= 1u << f;
        if (sn + 1 < nsteps) channels();  // the next launch forms its first step's anew
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
        if (f < p.nf)
#pragma unroll
            for (int m = 0; m < P; ++m) gstore(bufs.S[f] + dr + m * T, s[f][m]);
    if (bad) atomicOr(flag, bad);
    __syncthreads();  // every thread has read the counter
    if (advance && t == 0) *step_ctr += static_cast<uint64_t>(nsteps);
}

// The same for a line of one field whose only explicit term is one channel of
// products of that field, with operators in powers of q^2 (Model B, Model A):
// the state is kept as the N/2 + 1 modes k >= 0 of a real field, and both
// transforms are the complex ones of H = N/2 points on z[n] = x[2n] + i
// x[2n+1] (Van Loan, Sec. 4.3).  Against the kernel above that halves the
// noise (one Philox draw per mode and step, the largest part of its work),
// the update and the transforms.
//
// A thread keeps P of the H points, k = t + m T, in both transforms (natural
// order of modes, digit-reversed order of sites, which only meet pointwise
// products) and P/2 pairs of modes (k, H - k), k = t + m T < H/2, in between:
// the split into even and odd samples takes both of a pair, so the upper half
// of the points goes through an LDS line of H/2 on the way in and out, in
// which a thread reads and writes the same places.  Slot k = 0 holds modes 0
// and N/2 (both real) and, as its partner, H/2.
//
// One block on one CU is a serial chain: everything that a step does not
// change (operators, noise strengths, twiddles, the mask) is held in
// registers over the launch's steps, and lines up to 512 are one wave, with
// no barrier at all.  Four points a thread: 4096 (two waves a SIMD, 7800 of
// the 10000 cycles of a step issue vector instructions) took 4.2 us a step
// where 8 points took 4.4 and the kernel above 10.8; 1024: 2.4, 2.8 and 5.0; 64:
// 1.7 with 4 points, 4.4 with the kernel above.
template <int N>
__global__ void __launch_bounds__(line_half_threads(N) < 64 ? 64 : line_half_threads(N))
    line1d_half_kernel(const DevPlan* __restrict__ plan, Bufs bufs, uint64_t* __restrict__ step_ctr,
                       uint32_t* __restrict__ flag, int nsteps, int advance, const float2* __restrict__ tw_g) {
    constexpr int H = N / 2, P = kLineHalfPoints, PP = P / 2;
    using FFT = LineFFT<H, P>;
    constexpr int T = FFT::T;
    constexpr int NB = T < 64 ? T : 64;  // steps whose N/2 noise is drawn at once
    extern __shared__ float2 smem[];
    const DevPlan& p = *plan;
    const int t = threadIdx.x;
    LdsLine ld = FFT::lds_line(smem);
    float2* const xb = smem + FFT::kLds;

    const float dt = p.dt, inv_n = p.inv_n;
    const OpPoly imp = op_poly(p.implicit_op[0]), opc = op_poly(p.ch[0].op[0]), noi = op_poly(p.noise_op[0]);
    const bool noisy = p.noisy[0] != 0;
    const uint32_t key0 = p.key0, key1 = p.key1, fid = static_cast<uint32_t>(p.fid[0]);
    const int nprod = p.ch[0].nprod;
    const float coef0 = p.ch[0].prod[0].coef;
    const int pow0 = p.ch[0].prod[0].pow[0];
    const uint32_t step0 = static_cast<uint32_t>(gload_u64(step_ctr));
    const bool zero = t == 0;  // this thread's pair 0 is (0 and N/2, H/2)

    float2 a[PP], b[PP], wk[PP];
#pragma unroll
    for (int m = 0; m < PP; ++m) {
        const int k = t + m * T, kp = zero && m == 0 ? H / 2 : H - k;
        // Real space is the real part, whose mode k is the mean of phi(k) and
        // conj phi(-k): the modes themselves in a state that steps and uploads
        // leave, but not in any that a caller loads or writes
        const float2 ak = gload(bufs.S[0] + k), an = gload(bufs.S[0] + ((N - k) & (N - 1)));
        const float2 bk = gload(bufs.S[0] + kp), bn = gload(bufs.S[0] + N - kp);
        a[m] = make_float2(0.5f * (ak.x + an.x), 0.5f * (ak.y - an.y));
        b[m] = make_float2(0.5f * (bk.x + bn.x), 0.5f * (bk.y - bn.y));
        wk[m] = gload(tw_g + k);
    }
    if (zero) a[0].y = gload(bufs.S[0] + H).x;
    typename FFT::Regs tw;
    tw.load(tw_g, t, 2);

    // what the steps share: of the pair's modes, 1 / (1 - dt L), dt M / 2 (the
    // half of the split), the noise amplitude and the mask
    const DevMask mk = p.mask[0];
    auto q2_of = [&](int k) { return mode_q(p, k < (N >> 1) ? k : k - N, 0, 0).q2; };
    auto keep_of = [&](int k) { return mask_keep(mk, k < (N >> 1) ? k : k - N, 0, 0) ? 1.f : 0.f; };
    // rounded as in the other kernels: the factor's error repeats in every step
    auto implicit = [&](float q) { return cinv_implicit(dt, make_float2(horner(imp, q), 0.f)).x; };
    float ia[PP], ib[PP], ma[PP], mb[PP], na[PP], nb[PP], ka[PP], kb[PP];
#pragma unroll
    for (int m = 0; m < PP; ++m) {
        const int k = t + m * T, kp = zero && m == 0 ? H / 2 : H - k;
        const float qa = q2_of(k), qb = q2_of(kp);
        ia[m] = implicit(qa);
        ib[m] = implicit(qb);
        ma[m] = 0.5f * dt * horner(opc, qa);
        mb[m] = 0.5f * dt * horner(opc, qb);
        na[m] = p.amp_pair * __builtin_amdgcn_sqrtf(fmaxf(horner(noi, qa), 0.f));
        nb[m] = p.amp_pair * __builtin_amdgcn_sqrtf(fmaxf(horner(noi, qb), 0.f));
        ka[m] = keep_of(k);
        kb[m] = keep_of(kp);
    }
    // modes 0 and N/2 of slot 0
    const float qn = q2_of(H);
    const float n0 = p.amp_self * __builtin_amdgcn_sqrtf(fmaxf(horner(noi, q2_of(0)), 0.f));
    const float nn = p.amp_self * __builtin_amdgcn_sqrtf(fmaxf(horner(noi, qn), 0.f));
    const float in = implicit(qn), mn = 0.5f * dt * horner(opc, qn), kn = keep_of(H);

    auto draw = [&](uint32_t mode, uint32_t step) {
        const uint4 w = philox4x32_10(make_uint4(mode, step, fid, 0u), key0, key1);
        return box_muller(w.x, w.y);
    };
    // twice F[products] of the masked state at this thread's pairs
    float2 fa[PP], fb[PP];
    auto products = [&]() {
        float2 z[P];
#pragma unroll
        for (int m = 0; m < PP; ++m) {
            const float2 A = make_float2(a[m].x * ka[m], a[m].y * ka[m]), B = make_float2(b[m].x * kb[m], b[m].y * kb[m]);
            const float2 e = make_float2(A.x + B.x, A.y - B.y);                             // A + conj B
            const float2 o = cmul(make_float2(A.x - B.x, A.y + B.y), cconj(wk[m]));         // (A - conj B) / w
            float2 zl = make_float2(e.x - o.y, e.y + o.x), zh = make_float2(e.x + o.y, o.x - e.y);
            if (m == 0 && zero) {
                const float yn = a[0].y * kn;
                zl = make_float2(A.x + yn, A.x - yn);
                zh = make_float2(2.f * B.x, -2.f * B.y);
            }
            z[m] = zl;
            // k = 0: H/2, this thread's own first upper point
            xb[(H / 2 - t - m * T) & (H / 2 - 1)] = zh;
        }
        if constexpr (T > 64) __syncthreads(); else wave_lds_sync();
#pragma unroll
        for (int m = PP; m < P; ++m) z[m] = xb[t + (m - PP) * T];
        FFT::template dif<1>(z, ld, t, tw);
        // the products, even sites in .x and odd sites in .y
        float2 w[P];
#pragma unroll
        for (int m = 0; m < P; ++m) {
            z[m] = cscale(z[m], inv_n);
            w[m] = make_float2(coef0, coef0);
        }
        times_power<0>(w, z, pow0);
        for (int k = 1; k < nprod; ++k) {
            const DevProd& pd = p.ch[0].prod[k];
            float2 c[P];
#pragma unroll
            for (int m = 0; m < P; ++m) c[m] = make_float2(pd.coef, pd.coef);
            times_power<0>(c, z, pd.pow[0]);
#pragma unroll
            for (int m = 0; m < P; ++m) w[m] = cadd(w[m], c[m]);
        }
        FFT::template dit<-1>(w, ld, t, tw);
#pragma unroll
        for (int m = PP; m < P; ++m) xb[t + (m - PP) * T] = w[m];
        if constexpr (T > 64) __syncthreads(); else wave_lds_sync();
#pragma unroll
        for (int m = 0; m < PP; ++m) {
            const float2 zl = w[m], zh = xb[(H / 2 - t - m * T) & (H / 2 - 1)];
            const float2 e = make_float2(zl.x + zh.x, zl.y - zh.y);                 // 2 E = Z + conj Z'
            const float2 o = cmul(make_float2(zl.y + zh.y, zh.x - zl.x), wk[m]);    // 2 w O = -i w (Z - conj Z')
            fa[m] = cadd(e, o);
            fb[m] = make_float2(e.x - o.x, o.y - e.y);
            if (m == 0 && zero) {
                fa[0] = make_float2(2.f * (zl.x + zl.y), 2.f * (zl.x - zl.y));
                fb[0] = make_float2(2.f * zh.x, -2.f * zh.y);
            }
        }
    };

    float gn = 0.f;  // lane j: the normal of mode N/2 at step (sn & -NB) + j
    bool bad = false;
    for (int sn = 0; sn < nsteps; ++sn) {
        const uint32_t step = step0 + static_cast<uint32_t>(sn);
        products();
        if (noisy && (sn & (NB - 1)) == 0 && t < 64) gn = draw(H, step + static_cast<uint32_t>(t & (NB - 1))).x;
        const float gh = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gn), sn & (NB - 1)));
#pragma unroll
        for (int m = 0; m < PP; ++m) {
            const int k = t + m * T, kp = zero && m == 0 ? H / 2 : H - k;
            float2 ra = make_float2(fmaf(ma[m], fa[m].x, a[m].x), fmaf(ma[m], fa[m].y, a[m].y));
            float2 rb = make_float2(fmaf(mb[m], fb[m].x, b[m].x), fmaf(mb[m], fb[m].y, b[m].y));
            float ny = na[m], iy = ia[m];
            if (m == 0 && zero) {
                ra.y = fmaf(mn, fa[0].y, a[0].y);
                iy = in;
            }
            if (noisy) {
                float2 ga = draw(static_cast<uint32_t>(k), step);
                const float2 gb = draw(static_cast<uint32_t>(kp), step);
                float nx = na[m];
                if (m == 0 && zero) {
                    nx = n0;
                    ny = nn;
                    ga.y = gh;
                }
                ra = make_float2(fmaf(nx, ga.x, ra.x), fmaf(ny, ga.y, ra.y));
                rb = make_float2(fmaf(nb[m], gb.x, rb.x), fmaf(nb[m], gb.y, rb.y));
            }
            a[m] = make_float2(ra.x * ia[m], ra.y * iy);
            b[m] = cscale(rb, ib[m]);
            bad |= !(__builtin_isfinite(a[m].x) && __builtin_isfinite(a[m].y) && __builtin_isfinite(b[m].x) &&
                     __builtin_isfinite(b[m].y));
        }
    }
#pragma unroll
    for (int m = 0; m < PP; ++m) {
        const int k = t + m * T, kp = zero && m == 0 ? H / 2 : H - k;
        const bool z = zero && m == 0;
        gstore(bufs.S[0] + k, z ? make_float2(a[m].x, 0.f) : a[m]);
        gstore(bufs.S[0] + (z ? H : N - k), z ? make_float2(a[m].y, 0.f) : cconj(a[m]));
        gstore(bufs.S[0] + kp, b[m]);
        gstore(bufs.S[0] + N - kp, cconj(b[m]));
    }
    if (bad) atomicOr(flag, 1u);
    __syncthreads();  // every thread has read the counter
    if (advance && t == 0) *step_ctr += static_cast<uint64_t>(nsteps);
}

// This file is compiled once per line length with -DPSS_LINE_LEN=<L> (the
// kernels of that length) and once with -DPSS_COMMON (utilities and the
// length dispatch), so the instantiations build in parallel.
#if defined(PSS_LINE_LEN)
template <int L, int P, int NF, int DIM, bool TABLE>
static hipError_t launch_update_tab(int mode, const LaunchArgs& a, dim3 grid, dim3 block, size_t lds) {
#define PSS_UPD(M, G, NFV)                                                                                        \
    hipLaunchKernelGGL((update_kernel<L, P, NFV, M, DIM, G, TABLE>), grid, block, lds, a.stream, a.members, a.plans, \
                       a.plan, a.bufs, a.geo, a.step_ctr, a.flag, a.step_off, a.tw_u)
    switch (mode) {
        case MODE_STEP:
            if (a.general)
                PSS_UPD(MODE_STEP, true, NF);
            else
                PSS_UPD(MODE_STEP, false, NF);
            break;
        case MODE_PROLOGUE:
            if (a.general)
                PSS_UPD(MODE_PROLOGUE, true, NF);
            else
                PSS_UPD(MODE_PROLOGUE, false, NF);
            break;
        case MODE_INTERM_OUT: PSS_UPD(MODE_INTERM_OUT, true, NF); break;
        default: return hipErrorInvalidValue;
    }
#undef PSS_UPD
    return hipGetLastError();
}

template <int L, int P, int NF, int DIM>
static hipError_t launch_update_d(int mode, const LaunchArgs& a) {
    const int threads = a.geo.tc * a.geo.to * (L / P);
    const size_t lds = update_lds_bytes(L, P, a.geo.tc, a.geo.to);
    const bool tab = mode == MODE_STEP || mode == MODE_PROLOGUE || mode == MODE_INTERM_OUT;
    if (tab && (!a.members || !a.plans || a.nmem < 1)) return hipErrorInvalidValue;
    if (mode == MODE_INTERM_OUT && a.nmem != 1) return hipErrorInvalidValue;
    dim3 grid(a.geo.nublk, tab ? a.nmem : 1), block(threads);
    if (tab) {
        // one lattice: buffers, counter and flag come from the arguments
        if (a.nmem > 1) return launch_update_tab<L, P, NF, DIM, true>(mode, a, grid, block, lds);
        return launch_update_tab<L, P, NF, DIM, false>(mode, a, grid, block, lds);
    }
    switch (mode) {
        case MODE_FWD_STORE:
            hipLaunchKernelGGL((update_kernel<L, P, 1, MODE_FWD_STORE, DIM, false, false>), grid, block, lds, a.stream,
                               a.members, a.plans, a.plan, a.bufs, a.geo, a.step_ctr, a.flag, a.step_off, a.tw_u);
            break;
        case MODE_INV_OUT:
            hipLaunchKernelGGL((update_kernel<L, P, 1, MODE_INV_OUT, DIM, false, false>), grid, block, lds, a.stream,
                               a.members, a.plans, a.plan, a.bufs, a.geo, a.step_ctr, a.flag, a.step_off, a.tw_u);
            break;
        case MODE_FRAME_STEP:
        case MODE_FRAME_FWD:
            if constexpr (NF == 1 && DIM == 2) {
#define PSS_UF(M, G)                                                                                                \
    hipLaunchKernelGGL((update_kernel<L, P, 1, M, DIM, G, false>), grid, block, lds, a.stream, a.members, a.plans,  \
                       a.plan, a.bufs, a.geo, a.step_ctr, a.flag, a.step_off, a.tw_u)
                if (mode == MODE_FRAME_STEP) {
                    if (a.general)
                        PSS_UF(MODE_FRAME_STEP, true);
                    else
                        PSS_UF(MODE_FRAME_STEP, false);
                } else {
                    if (a.general)
                        PSS_UF(MODE_FRAME_FWD, true);
                    else
                        PSS_UF(MODE_FRAME_FWD, false);
                }
#undef PSS_UF
                break;
            }
            return hipErrorInvalidValue;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int L, int P, int NF>
static hipError_t launch_update_t(int mode, const LaunchArgs& a) {
    return a.dim == 3 ? launch_update_d<L, P, NF, 3>(mode, a) : launch_update_d<L, P, NF, 2>(mode, a);
}

template <int L, int P, int NG>
static hipError_t launch_xrow_t(int mode, const LaunchArgs& a) {
    const int threads = (a.geo.rb / 2) * (L / P);
    const size_t lds = xrow_lds_bytes(L, P, a.geo.rb);
    const bool tab = mode == MODE_STEP;
    if (tab && (!a.members || !a.plans || a.nmem < 1)) return hipErrorInvalidValue;
    dim3 grid(a.geo.nrowblk, tab ? a.nmem : 1), block(threads);
    uint64_t* ctr = const_cast<uint64_t*>(a.step_ctr);
    switch (mode) {
        case MODE_STEP:
            if (a.nmem > 1)
                hipLaunchKernelGGL((xrow_kernel<L, P, NG, MODE_STEP, true>), grid, block, lds, a.stream, a.members,
                                   a.plans, a.plan, a.bufs, a.geo, a.tw_x, a.advance, ctr);
            else
                hipLaunchKernelGGL((xrow_kernel<L, P, NG, MODE_STEP, false>), grid, block, lds, a.stream, a.members,
                                   a.plans, a.plan, a.bufs, a.geo, a.tw_x, a.advance, ctr);
            break;
        case MODE_R2C_IN:
            hipLaunchKernelGGL((xrow_kernel<L, P, 1, MODE_R2C_IN, false>), grid, block, lds, a.stream, a.members,
                               a.plans, a.plan, a.bufs, a.geo, a.tw_x, int64_t{0}, ctr);
            break;
        case MODE_C2R_OUT:
            hipLaunchKernelGGL((xrow_kernel<L, P, 1, MODE_C2R_OUT, false>), grid, block, lds, a.stream, a.members,
                               a.plans, a.plan, a.bufs, a.geo, a.tw_x, int64_t{0}, ctr);
            break;
        case MODE_FRAME_ROW:
            if (a.geo.nz != 1 || !a.bufs.frame_rows) return hipErrorInvalidValue;
            hipLaunchKernelGGL((xrow_kernel<L, P, 1, MODE_FRAME_ROW, false>), grid, block, lds, a.stream, a.members,
                               a.plans, a.plan, a.bufs, a.geo, a.tw_x, int64_t{0}, ctr);
            break;
        case MODE_ADJROW:
            if ((threads & 63) != 0 && threads > 64) return hipErrorInvalidValue;  // block_sum_to_slot's shapes
            if constexpr (NG == 2) {
                hipLaunchKernelGGL((xrow_kernel<L, P, 2, MODE_ADJROW, false>), grid, block, lds, a.stream, a.members,
                                   a.plans, a.plan, a.bufs, a.geo, a.tw_x, int64_t{0}, ctr);
                break;
            }
            return hipErrorInvalidValue;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define PSS_CAT2(a, b) a##b
#define PSS_CAT(a, b) PSS_CAT2(a, b)

// points-per-thread variants: P = geo.pu (update) or geo.px (x kernel), any
// of 16, 8, 4 not above the cap for the number of register arrays
template <int L, int CAP, class F>
static hipError_t with_points(int want, F&& f) {
    if constexpr (L >= 16 && CAP >= 16) {
        if (want == 16) return f(std::integral_constant<int, 16>{});
    }
    if constexpr (L >= 8 && CAP >= 8) {
        if (want == 8) return f(std::integral_constant<int, 8>{});
    }
    if constexpr (L >= 4 && CAP >= 4) {
        if (want == 4) return f(std::integral_constant<int, 4>{});
    }
    if constexpr (L < 4) {
        if (want == L) return f(std::integral_constant<int, L>{});
    }
    return hipErrorInvalidValue;
}

template <int NF, bool GEN>
static hipError_t launch_line1d_t(int mode, const LaunchArgs& a) {
    constexpr int N = PSS_LINE_LEN;
    const dim3 grid(1), block(N / 4);
    const size_t lds = line1d_lds_bytes(N);
    uint64_t* ctr = const_cast<uint64_t*>(a.step_ctr);
    if constexpr (NF == 1 && !GEN) {
        if (mode == MODE_STEP && a.simple && !a.framed) {
            hipLaunchKernelGGL((line1d_half_kernel<N>), grid, dim3(line_half_threads(N)), line_half_lds_bytes(N), a.stream,
                               a.plan, a.bufs, ctr, a.flag, a.nsteps, a.advance != 0 ? 1 : 0, a.tw_x);
            return hipGetLastError();
        }
    }
#define PSS_L1(M)                                                                                                 \
    hipLaunchKernelGGL((line1d_kernel<N, NF, GEN, M>), grid, block, lds, a.stream, a.plan, a.bufs, ctr, a.flag, \
                       a.nsteps, a.advance != 0 ? 1 : 0, a.tw_x)
    switch (mode) {
        case MODE_STEP: PSS_L1(MODE_STEP); break;
        case MODE_FWD_STORE: PSS_L1(MODE_FWD_STORE); break;
        case MODE_INV_OUT: PSS_L1(MODE_INV_OUT); break;
        case MODE_INTERM_OUT: PSS_L1(MODE_INTERM_OUT); break;
        default: return hipErrorInvalidValue;
    }
#undef PSS_L1
    return hipGetLastError();
}

hipError_t PSS_CAT(launch_line1d_L, PSS_LINE_LEN)(int mode, int nf, const LaunchArgs& a) {
    if (mode == MODE_FWD_STORE || mode == MODE_INV_OUT) return launch_line1d_t<1, false>(mode, a);
    const bool gen = a.general || mode == MODE_INTERM_OUT;
    if (nf <= 1) return gen ? launch_line1d_t<1, true>(mode, a) : launch_line1d_t<1, false>(mode, a);
    if (nf == 2) return gen ? launch_line1d_t<2, true>(mode, a) : launch_line1d_t<2, false>(mode, a);
    if (nf <= 4) return gen ? launch_line1d_t<4, true>(mode, a) : launch_line1d_t<4, false>(mode, a);
    return hipErrorInvalidValue;
}

hipError_t PSS_CAT(line1d_setup_L, PSS_LINE_LEN)() {
    constexpr int N = PSS_LINE_LEN;
    const int lds = static_cast<int>(line1d_lds_bytes(N));
#define PSS_L1A(NFV, G, M)                                                                                       \
    if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&line1d_kernel<N, NFV, G, M>),          \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds))                     \
        return e;
#define PSS_L1B(M) PSS_L1A(1, false, M) PSS_L1A(1, true, M) PSS_L1A(2, false, M) PSS_L1A(2, true, M) \
    PSS_L1A(4, false, M) PSS_L1A(4, true, M)
    PSS_L1B(MODE_STEP)
    PSS_L1B(MODE_INTERM_OUT)
    PSS_L1A(1, false, MODE_FWD_STORE)
    PSS_L1A(1, false, MODE_INV_OUT)
#undef PSS_L1B
#undef PSS_L1A
    return hipSuccess;
}

hipError_t PSS_CAT(launch_update_L, PSS_LINE_LEN)(int mode, int nf, const LaunchArgs& a) {
    constexpr int L = PSS_LINE_LEN;
    const int pu = a.geo.pu;
    if (mode == MODE_FWD_STORE || mode == MODE_INV_OUT || nf <= 1)
        return with_points<L, 16>(pu, [&](auto P) { return launch_update_t<L, decltype(P)::value, 1>(mode, a); });
    if (nf == 2)
        return with_points<L, 8>(pu, [&](auto P) { return launch_update_t<L, decltype(P)::value, 2>(mode, a); });
    if (nf <= 4)
        return with_points<L, 4>(pu, [&](auto P) { return launch_update_t<L, decltype(P)::value, 4>(mode, a); });
    return hipErrorInvalidValue;
}

hipError_t PSS_CAT(launch_ypass_L, PSS_LINE_LEN)(int mode, const YArgs& ya, const LaunchArgs& a) {
    constexpr int L = PSS_LINE_LEN;
    return with_points<L, 16>(a.geo.py, [&](auto PP) {
        constexpr int P = decltype(PP)::value;
        const int threads = a.geo.tc * a.geo.tz * (L / P);
        const size_t lds = ypass_lds_bytes(L, P, a.geo.tc, a.geo.tz);
        dim3 grid(a.geo.nyblk), block(threads);
        if (mode == MODE_YINV) {
            hipLaunchKernelGGL((ypass_kernel<L, P, MODE_YINV>), grid, block, lds, a.stream, ya, a.geo, a.tw_y);
        } else if (mode == MODE_YFWD) {
            hipLaunchKernelGGL((ypass_kernel<L, P, MODE_YFWD>), grid, block, lds, a.stream, ya, a.geo, a.tw_y);
        } else {
            return hipErrorInvalidValue;
        }
        return hipGetLastError();
    });
}

hipError_t PSS_CAT(launch_adjcol_L, PSS_LINE_LEN)(int mode, const AdjArgs& aa, const LaunchArgs& a) {
    constexpr int L = PSS_LINE_LEN;
    return with_points<L, 16>(a.geo.pu, [&](auto PP) {
        constexpr int P = decltype(PP)::value;
        const int threads = a.geo.tc * (L / P);
        const size_t lds = update_lds_bytes(L, P, a.geo.tc, 1);
        dim3 grid(a.geo.nublk), block(threads);
        if (a.dim != 2 || a.geo.to != 1) return hipErrorInvalidValue;
        if ((threads & 63) != 0 && threads > 64) return hipErrorInvalidValue;  // block_sum_to_slot's shapes
        if (mode == MODE_ADJCOL) {
            hipLaunchKernelGGL((adjcol_kernel<L, P, MODE_ADJCOL>), grid, block, lds, a.stream, aa, a.geo, a.tw_u);
        } else if (mode == MODE_ADJFIN) {
            hipLaunchKernelGGL((adjcol_kernel<L, P, MODE_ADJFIN>), grid, block, lds, a.stream, aa, a.geo, a.tw_u);
        } else {
            return hipErrorInvalidValue;
        }
        return hipGetLastError();
    });
}

hipError_t PSS_CAT(launch_xrow_L, PSS_LINE_LEN)(int mode, int ng, const LaunchArgs& a) {
    constexpr int L = PSS_LINE_LEN;
    const int px = a.geo.px;
    if ((mode != MODE_STEP && mode != MODE_ADJROW) || ng <= 1)
        return with_points<L, 16>(px, [&](auto P) { return launch_xrow_t<L, decltype(P)::value, 1>(mode, a); });
    if (ng == 2)
        return with_points<L, 8>(px, [&](auto P) { return launch_xrow_t<L, decltype(P)::value, 2>(mode, a); });
    if (ng == 3)
        return with_points<L, 4>(px, [&](auto P) { return launch_xrow_t<L, decltype(P)::value, 3>(mode, a); });
    if (ng == 4)
        return with_points<L, 4>(px, [&](auto P) { return launch_xrow_t<L, decltype(P)::value, 4>(mode, a); });
    if (mode != MODE_STEP) return hipErrorInvalidValue;
    // five to eight factor slots (multi-field flow models): one variant with
    // room for eight, 4 points per thread
    if (ng <= PSS_MAXG)
        return with_points<L, 4>(px, [&](auto P) { return launch_xrow_t<L, decltype(P)::value, PSS_MAXG>(mode, a); });
    return hipErrorInvalidValue;
}
#endif  // PSS_LINE_LEN

#if defined(PSS_BATCH)
// ------------------------------------------------------ fused batch launches
// One launch per phase for a whole batch: block b (XCD-ordered) finds its
// class in the work list, then its member and tile, and runs the block body
// built for that class's line length.
__device__ __forceinline__ int batch_class_of(const BatchLaunch& bl, int b) {
    int k = 0;
    for (int i = 1; i < bl.ncls; ++i)
        if (b >= bl.cls[i].start) k = i;
    return k;
}

__global__ void __launch_bounds__(256) batch_update_kernel(BatchLaunch bl) {
    // uniform by construction; said so, since the division runs on the VALU
    const int b = __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x));
    const BatchClass& C = bl.cls[__builtin_amdgcn_readfirstlane(batch_class_of(bl, b))];
    const int rel = b - C.start;
    const int mi = __builtin_amdgcn_readfirstlane(rel / C.nblk);
    const int blk = rel - mi * C.nblk;
    const Bufs none{};
#define PSS_BU(LL)                                                                                                 \
    case LL:                                                                                                       \
        update_block<LL, 4, 1, MODE_STEP, 2, false, true>(mi, blk, C.members, C.plans, nullptr, none, C.geo,       \
                                                             nullptr,                                                 \
                                                          nullptr, bl.step_off, C.tw);                             \
        break;
    switch (C.L) {
        PSS_BU(64)
        PSS_BU(128)
        PSS_BU(256)
        PSS_BU(512)
        PSS_BU(1024)
        default: break;
    }
#undef PSS_BU
}

__global__ void __launch_bounds__(256) batch_xrow_kernel(BatchLaunch bl) {
    // uniform by construction; said so, since the division runs on the VALU
    const int b = __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x));
    const BatchClass& C = bl.cls[__builtin_amdgcn_readfirstlane(batch_class_of(bl, b))];
    const int rel = b - C.start;
    const int mi = __builtin_amdgcn_readfirstlane(rel / C.nblk);
    const int blk = rel - mi * C.nblk;
    const Bufs none{};
#define PSS_BX(LL)                                                                                          \
    case LL:                                                                                                \
        xrow_block<LL, 4, 1, MODE_STEP, true>(mi, blk, C.members, C.plans, nullptr, none, C.geo, C.tw, bl.advance, \
                                              nullptr);                                                     \
        break;
    switch (C.L) {
        PSS_BX(64)
        PSS_BX(128)
        PSS_BX(256)
        PSS_BX(512)
        PSS_BX(1024)
        default: break;
    }
#undef PSS_BX
}

// ------------------------------------------------- LDS-resident multi-step
// One block holds a whole lattice: its state in registers (each thread keeps
// the slots of its column lines), the channel and factor arrays in one LDS
// array X[c][position] (column stride Ny + 1), which each phase overwrites in
// place: the column phase reads a column's channel values and writes its
// factor values, the row phase reads a row pair's factor values and writes
// its channel values.  The two phases are the update kernel's and the x
// kernel's line bodies with LDS in place of the packed-column arrays: the
// same transforms (4 points per thread; every line fits in a wave, so only
// the packed line's exchange and the phase changes take block barriers), the
// same operations in the same order, and the same position order of the
// exchanged arrays (the x phase works on positions as rows).  The launch
// loads the state and the channel array, runs rl.nsteps steps, stores both
// back and moves the member's step counter on.
//
// What bounds it: one block of 16 waves a CU, so 128 registers a thread, 70 %
// of whose cycles issue vector instructions at 128^2.  The plan's values stay
// in scalar registers and the twiddles in vector registers over the steps
// (they were read from memory and from LDS in each), and addresses and q^2 are
// formed where they are used: hoisted out of the loop over steps they spilled.
// 256 lattices, a step: 128^2 23.2 -> 20.0 us, 64 x 128 12.5 -> 10.8, 64^2 9.4
// -> 6.6.
template <int LX, int LY>
__global__ void __launch_bounds__(resident_threads(LX, LY)) resident_kernel(ResidentLaunch rl) {
    constexpr int P = 4;
    using FY = LineFFT<LY, P>;
    using FX = LineFFT<LX, P>;
    static_assert(!FY::kCross && !FX::kCross, "lines held by one wave");
    constexpr int TY = FY::T, TX = FX::T;
    constexpr int NC = LX / 2;                      // packed columns
    constexpr int NTHR = resident_threads(LX, LY);
    constexpr int CPR = NTHR / TY, RPR = NTHR / TX;  // column lines, row pairs per round
    constexpr int CR = NC / CPR;                     // rounds of each phase
    static_assert(CR * CPR == NC && CR * RPR == LY / 2, "whole rounds");
    constexpr int XS = LY + 1;                       // column stride of X
    constexpr int LPW = 64 / TY;                     // column lines per wave
    extern __shared__ float2 smem[];
    float2* const X = smem;
    float2* const scr = X + NC * XS;                 // one exchange region per line of a round
    constexpr int SCR = CPR * FY::kReg > RPR * FX::kReg ? CPR * FY::kReg : RPR * FX::kReg;
    float2* const xbuf = scr + SCR;                  // packed-line exchange (LY)
    const int mi = __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x));
    const Member& mem = rl.members[mi];
    const DevPlan& p = rl.plans[mi];
    const int tid = threadIdx.x;
    const int tc = rl.geo.tc, lt = rl.geo.tc_log2;
    const int nx = p.n[0];
    float2* __restrict__ Sg = mem.bufs.S[0];
    float2* __restrict__ Ng = mem.bufs.N[0];

    // column phase: line li of the round, thread t of the line
    const int li = tid / TY, tcol = tid & (TY - 1);
    LdsLine ldc;
    ldc.wl = scr + li * FY::kReg;
    ldc.blk0 = ldc.blk1 = nullptr;
    ldc.par = 0;
    // row phase: pair pi of the round, thread t of the pair
    const int pi = tid / TX, trow = tid & (TX - 1);
    LdsLine ldr;
    ldr.wl = scr + pi * FX::kReg;
    ldr.blk0 = ldr.blk1 = nullptr;
    ldr.par = 0;

    // twiddles: 6 or 8 values, the same for both directions of a square lattice
    typename FY::Regs twy;
    typename FX::Regs twx_own;
    twy.load(rl.tw_y, tcol);
    if constexpr (LX != LY) twx_own.load(rl.tw_x, trow);
    const auto& twx = [&]() -> const auto& {
        if constexpr (LX == LY)
            return twy;
        else
            return twx_own;
    }();
    // the state of this thread's column slots, and the channel array
    float2 st[CR][P];
#pragma unroll
    for (int r = 0; r < CR; ++r) {
        const int c = r * CPR + li;
        const size_t base = (static_cast<size_t>(c >> lt) * LY << lt) + (c & (tc - 1));
#pragma unroll
        for (int m = 0; m < P; ++m) st[r][m] = gload(Sg + base + static_cast<size_t>(tcol + m * TY) * tc);
    }
    // place in X of element i of the channel array, which lies as the step
    // kernels' exchange arrays do (Exch): column tiles, or groups of four rows
    const bool grp = rl.geo.grp != 0;
    auto place = [&](int i) {
        if (grp) {
            const int g = i >> 2;
            return (g & (NC - 1)) * XS + 4 * (g / NC) + (i & 3);
        }
        const int ct = i / (LY * tc), rem = i - ct * (LY * tc);
        return ((ct << lt) + (rem & (tc - 1))) * XS + (rem >> lt);
    };
    for (int i = tid; i < NC * LY; i += NTHR) X[place(i)] = gload(Ng + i);
    const uint32_t step0 = static_cast<uint32_t>(gload_u64(mem.step_ctr));
    // the plan's values, once for all steps
    float dt = p.dt, qs[3] = {p.qs[0], p.qs[1], p.qs[2]}, inv_n = p.inv_n, amp_pair = p.amp_pair, amp_self = p.amp_self;
    uint32_t key0 = p.key0, key1 = p.key1;
    int noisy = p.noisy[0], fid = p.fid[0], nch = p.nch, nd = p.nd, ng = p.ng, ncol = p.mask[0].ncol, ny = p.n[1];
    OpPoly imp = op_poly(p.implicit_op[0]), noi = op_poly(p.noise_op[0]), ch0 = op_poly(p.ch[0].op[0]);
    hold(dt), hold(inv_n), hold(amp_pair), hold(amp_self), hold(key0), hold(key1), hold(noisy), hold(fid), hold(nch);
    hold(nd), hold(ng), hold(ncol), hold(ny), hold(imp), hold(noi), hold(ch0);
#pragma unroll
    for (int i = 0; i < 3; ++i) hold(qs[i]);
    // the four self-conjugate modes of column 0, one per lane (as in the update kernel)
    const Self self = self_modes<LY, 2>(nx, LY, 1, qs, 0, tid);
    __syncthreads();

    uint32_t bad = 0;
    for (int sn = 0; sn < rl.nsteps; ++sn) {
        const uint32_t step = step0 + static_cast<uint32_t>(sn);
        const NoiseKey nk{key0, key1, step, fid, amp_pair, amp_self};
        // ---- column phase: forward y transform of the channel, update,
        // de-aliased inverse y transform of the factor
#pragma unroll
        for (int r = 0; r < CR; ++r) {
            int lif = li;
            fresh(lif);
            const int c = r * CPR + lif;
            const bool blk_packed = r == 0;  // the round holding column 0 (block-uniform)
            const bool packed = c == 0;
            const bool pair_lane = packed && tcol == 0;
            const bool first_wave = blk_packed && tid < 64;
            const int kx_l = c, ky_l = 0;
            float2* const col = X + c * XS;
            auto exchange = [&](float2 (&v)[P], bool forward) {
                if (!blk_packed) return;
                if (packed) {
#pragma unroll
                    for (int m = 0; m < P; ++m) xbuf[tcol + m * TY] = v[m];
                }
                __syncthreads();
                if (packed) {
#pragma unroll
                    for (int m = 0; m < P; ++m) {
                        const int u = tcol + m * TY;
                        const float2 b = xbuf[(LY - u) & (LY - 1)];
                        v[m] = forward ? to_slot<LY>(u, v[m], b) : from_slot<LY>(u, v[m], b);
                    }
                }
                __syncthreads();
            };
            const LineModes lmode = line_modes<LY, 2>(nx, ny, qs, packed, kx_l, ky_l);
            float2(&s)[P] = st[r];
            // one round after the other, and within it one thing after the
            // other: interleaved, they spilled
            __builtin_amdgcn_sched_barrier(0);
            auto slot_q2 = [&](float (&q2)[P]) {
                int tq = tcol;
                fresh(tq);
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    uint32_t lin, lneg;
                    slot_at<LY>(lmode, tq + m * TY, q2[m], lin, lneg);
                }
            };
            float2 acc[P];
#pragma unroll
            for (int m = 0; m < P; ++m) acc[m] = make_float2(0.f, 0.f);
            auto add_term = [&](const OpPoly& op, const float2 (&v)[P]) {
                float q2[P], M[P];
                slot_q2(q2);
                horner_p(op, q2, M);
                Four f{};
                if (first_wave) f = four_lanes(horner(op, self.q.q2));
#pragma unroll
                for (int m = 0; m < P; ++m)
                    if (!(pair_lane && (m == 0 || m == P / 2))) acc[m] = cadd(acc[m], cscale(v[m], M[m]));
                if (pair_lane) {
                    float2 lo, hi;
                    pair_scale(f, v, lo, hi);
                    acc[0] = cadd(acc[0], lo);
                    acc[P / 2] = cadd(acc[P / 2], hi);
                }
            };
            if (nch > 0) {
                float2 v[P];
#pragma unroll
                for (int m = 0; m < P; ++m) v[m] = col[tcol + m * TY];
                FY::template dit<-1>(v, ldc, tcol, twy);
                exchange(v, true);
                add_term(ch0, v);
            }
            for (int d = 0; d < nd; ++d) add_term(op_poly(p.direct[d].op), s);
            {
#pragma unroll
                for (int m = 0; m < P; ++m) s[m] = cadd(s[m], cscale(acc[m], dt));
                const float2 old0 = s[0], oldh = s[P / 2];
                __builtin_amdgcn_sched_barrier(0);
                float q2[P], A[P];
                slot_q2(q2);
                if (noisy) {
                    int tq = tcol;
                    fresh(tq);
                    horner_p(noi, q2, A);
#pragma unroll
                    for (int m = 0; m < P; ++m) {
                        float q2m;
                        uint32_t lin, lneg;
                        slot_at<LY>(lmode, tq + m * TY, q2m, lin, lneg);
                        s[m] = cadd(s[m], noise_value<true>(nk, lin, lneg, A[m]));
                        if (m & 1) __builtin_amdgcn_sched_barrier(0);
                    }
                }
                horner_p(imp, q2, A);
#pragma unroll
                for (int m = 0; m < P; ++m) s[m] = cscale(s[m], __builtin_amdgcn_rcpf(fmaf(-dt, A[m], 1.f)));
                if (first_wave) {
                    const Four inv = four_lanes(cinv_implicit(dt, make_float2(horner(imp, self.q.q2), 0.f)).x);
                    Four e{};
                    if (noisy) e = four_lanes(noise_value(nk, self.lin, self.lneg, horner(noi, self.q.q2)).x);
                    if (pair_lane) {
                        float2 rl = old0, rh = oldh;
                        if (noisy) {
                            rl = make_float2(rl.x + e.v[0], rl.y + e.v[1]);
                            rh = make_float2(rh.x + e.v[2], rh.y + e.v[3]);
                        }
                        pair_scale<2>(inv, {rl, rh}, s[0], s[P / 2]);
                    }
                }
                bool fin = true;
#pragma unroll
                for (int m = 0; m < P; ++m) fin = fin && __builtin_isfinite(s[m].x) && __builtin_isfinite(s[m].y);
                if (!fin) bad |= 1u;
            }
            // de-aliased inverse transform of the factor (lines of a wave whose
            // first column is past the kept ones are never read)
            if (ng > 0 && (c / LPW) * LPW < ncol) {
                const int lim = p.lim[0][kx_l], limN = p.lim[0][nx >> 1];
                float2 v[P];
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    const int u = tcol + m * TY;
                    const bool upper = packed && u > (LY >> 1);
                    const int w = packed ? (upper ? LY - u : u) : (u < (LY >> 1) ? u : u - LY);
                    v[m] = w * w <= (upper ? limN : lim) ? s[m] : make_float2(0.f, 0.f);
                }
                if (pair_lane) {
                    const int wh = (LY >> 1) * (LY >> 1);
                    const float2 a0 = s[0], ah = s[P / 2];
                    v[0] = make_float2(0 <= lim ? a0.x : 0.f, 0 <= limN ? a0.y : 0.f);
                    v[P / 2] = make_float2(wh <= lim ? ah.x : 0.f, wh <= limN ? ah.y : 0.f);
                }
                exchange(v, false);
                FY::template dif<1>(v, ldc, tcol, twy);
#pragma unroll
                for (int m = 0; m < P; ++m) col[tcol + m * TY] = v[m];
            } else if (blk_packed) {
                // the packed line's exchange barriers are block-wide
                __syncthreads();
                __syncthreads();
            }
        }
        __syncthreads();
        // ---- row phase: inverse x transform of each row pair's factor
        // values, the products, forward x transform into the channel values
#pragma unroll
        for (int r = 0; r < CR; ++r) {
            int pf = pi, tf = trow;
            fresh(pf);
            fresh(tf);
            const int p0 = 2 * (r * RPR + pf);  // first position of the pair
            if (nch == 0) break;
            __builtin_amdgcn_sched_barrier(0);
            float2 v[P];
            {
                float2 a[P], b[P];
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    const int k = tf + m * TX;
                    const int kk = (k == NC) ? 0 : (k < NC ? k : LX - k);
                    const int kc = kk < ncol ? kk : 0;
                    a[m] = X[kc * XS + p0];
                    b[m] = X[kc * XS + p0 + 1];
                }
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    const int k = tf + m * TX;
                    const int kk = (k == NC) ? 0 : (k < NC ? k : LX - k);
                    const float2 zero = make_float2(0.f, 0.f);
                    const float2 am = kk < ncol ? a[m] : zero, bm = kk < ncol ? b[m] : zero;
                    float2 z;
                    if (k == 0) {
                        z = make_float2(am.x, bm.x);
                    } else if (k == NC) {
                        z = make_float2(am.y, bm.y);
                    } else {
                        z = k < NC ? make_float2(am.x - bm.y, am.y + bm.x) : make_float2(am.x + bm.y, bm.x - am.y);
                    }
                    v[m] = z;
                }
            }
            FX::template dif<1>(v, ldr, trow, twx);
            float2 z[P];
#pragma unroll
            for (int m = 0; m < P; ++m) z[m] = cscale(v[m], inv_n);
            const DevChannel& C = p.ch[0];
            float2 w[P];
#pragma unroll
            for (int m = 0; m < P; ++m) w[m] = make_float2(0.f, 0.f);
            for (int k = 0; k < C.nprod; ++k) {
                const DevProd& pd = C.prod[k];
                const int pg = static_cast<int>(pd.pow[0]);
                float2 a[P];
#pragma unroll
                for (int m = 0; m < P; ++m) a[m] = make_float2(pd.coef, pd.coef);
                times_power<0>(a, z, pg);
#pragma unroll
                for (int m = 0; m < P; ++m) w[m] = cadd(w[m], a[m]);
            }
            FX::template dit<-1>(w, ldr, trow, twx);
            // unpack the pair's two rows into the packed columns
            float2* const W = ldr.wl;
            wave_lds_sync();
#pragma unroll
            for (int m = 0; m < P; ++m) W[trow + m * TX] = w[m];
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < NC / TX; ++j) {
                const int c = tf + j * TX;
#pragma unroll
                for (int rr = 0; rr < 2; ++rr) {
                    float2 o;
                    if (c == 0) {
                        const float2 a = W[0], b = W[NC];
                        o = rr ? make_float2(a.y, b.y) : make_float2(a.x, b.x);
                    } else {
                        const float2 a = W[c], b = W[LX - c];
                        o = rr ? make_float2(0.5f * (a.y + b.y), 0.5f * (b.x - a.x))
                               : make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
                    }
                    X[c * XS + p0 + rr] = o;
                }
            }
        }
        __syncthreads();
    }

    // state and channel array back to HBM; the counter moves on
#pragma unroll
    for (int r = 0; r < CR; ++r) {
        const int c = r * CPR + li;
        const size_t base = (static_cast<size_t>(c >> lt) * LY << lt) + (c & (tc - 1));
#pragma unroll
        for (int m = 0; m < P; ++m) gstore(Sg + base + static_cast<size_t>(tcol + m * TY) * tc, st[r][m]);
    }
    for (int i = tid; i < NC * LY; i += NTHR) gstore(Ng + i, X[place(i)]);
    if (bad) atomicOr(mem.flag, bad);
    if (rl.advance && tid == 0) *mem.step_ctr += static_cast<uint64_t>(rl.nsteps);
}

// allow the resident kernels their LDS (above the default dynamic limit)
hipError_t resident_setup() {
#define PSS_RES_ATTR(AX, AY)                                                                                     \
    if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&resident_kernel<AX, AY>),              \
                                           hipFuncAttributeMaxDynamicSharedMemorySize,                            \
                                           static_cast<int>(resident_lds_bytes(AX, AY))))                        \
        return e;
    PSS_RES_ATTR(64, 64)
    PSS_RES_ATTR(64, 128)
    PSS_RES_ATTR(128, 64)
    PSS_RES_ATTR(128, 128)
#undef PSS_RES_ATTR
    return hipSuccess;
}

hipError_t launch_batch_resident(hipStream_t s, const ResidentLaunch& rl) {
    if (rl.nmem < 1 || rl.nsteps < 1) return hipSuccess;
    const size_t lds = resident_lds_bytes(rl.lx, rl.ly);
#define PSS_RES(AX, AY)                                                                                      if (rl.lx == AX && rl.ly == AY) {                                                                            hipLaunchKernelGGL((resident_kernel<AX, AY>), dim3(rl.nmem), dim3(resident_threads(AX, AY)), lds, s, rl);         return hipGetLastError();                                                                            }
    PSS_RES(64, 64)
    PSS_RES(64, 128)
    PSS_RES(128, 64)
    PSS_RES(128, 128)
#undef PSS_RES
    return hipErrorInvalidValue;
}

hipError_t launch_batch_update(hipStream_t s, const BatchLaunch& bl, size_t lds) {
    if (bl.ncls < 1 || bl.total < 1) return hipSuccess;
    hipLaunchKernelGGL(batch_update_kernel, dim3(bl.total), dim3(256), lds, s, bl);
    return hipGetLastError();
}

hipError_t launch_batch_xrow(hipStream_t s, const BatchLaunch& bl, size_t lds) {
    if (bl.ncls < 1 || bl.total < 1) return hipSuccess;
    hipLaunchKernelGGL(batch_xrow_kernel, dim3(bl.total), dim3(256), lds, s, bl);
    return hipGetLastError();
}
#endif  // PSS_BATCH

#if defined(PSS_COMMON)
#define PSS_DECL_L(L)                                                               \
    hipError_t launch_line1d_L##L(int mode, int nf, const LaunchArgs& a);          \
    hipError_t line1d_setup_L##L();                                                 \
    hipError_t launch_update_L##L(int mode, int nf, const LaunchArgs& a);          \
    hipError_t launch_ypass_L##L(int mode, const YArgs& ya, const LaunchArgs& a);  \
    hipError_t launch_xrow_L##L(int mode, int ng, const LaunchArgs& a);            \
    hipError_t launch_adjcol_L##L(int mode, const AdjArgs& aa, const LaunchArgs& a);
PSS_DECL_L(8)
PSS_DECL_L(16)
PSS_DECL_L(32)
PSS_DECL_L(64)
PSS_DECL_L(128)
PSS_DECL_L(256)
PSS_DECL_L(512)
PSS_DECL_L(1024)
PSS_DECL_L(2048)
PSS_DECL_L(4096)

int max_points(int L, int nregs) {
    const int cap = nregs <= 1 ? 16 : (nregs == 2 ? 8 : 4);
    return cap < L ? cap : L;
}

hipError_t launch_line1d(int mode, int N, int nf, const LaunchArgs& a) {
    switch (N) {
        case 8: return launch_line1d_L8(mode, nf, a);
        case 16: return launch_line1d_L16(mode, nf, a);
        case 32: return launch_line1d_L32(mode, nf, a);
        case 64: return launch_line1d_L64(mode, nf, a);
        case 128: return launch_line1d_L128(mode, nf, a);
        case 256: return launch_line1d_L256(mode, nf, a);
        case 512: return launch_line1d_L512(mode, nf, a);
        case 1024: return launch_line1d_L1024(mode, nf, a);
        case 2048: return launch_line1d_L2048(mode, nf, a);
        case 4096: return launch_line1d_L4096(mode, nf, a);
        default: return launch_line1d_mr(mode, N, nf, a.ng, a);
    }
}

hipError_t line1d_setup(int N) {
    switch (N) {
        case 8: return line1d_setup_L8();
        case 16: return line1d_setup_L16();
        case 32: return line1d_setup_L32();
        case 64: return line1d_setup_L64();
        case 128: return line1d_setup_L128();
        case 256: return line1d_setup_L256();
        case 512: return line1d_setup_L512();
        case 1024: return line1d_setup_L1024();
        case 2048: return line1d_setup_L2048();
        case 4096: return line1d_setup_L4096();
        default: return line1d_mr_setup();
    }
}

hipError_t launch_update(int mode, int L, int nf, const LaunchArgs& a) {
    switch (L) {
        case 8: return launch_update_L8(mode, nf, a);
        case 16: return launch_update_L16(mode, nf, a);
        case 32: return launch_update_L32(mode, nf, a);
        case 64: return launch_update_L64(mode, nf, a);
        case 128: return launch_update_L128(mode, nf, a);
        case 256: return launch_update_L256(mode, nf, a);
        case 512: return launch_update_L512(mode, nf, a);
        case 1024: return launch_update_L1024(mode, nf, a);
        case 2048: return launch_update_L2048(mode, nf, a);
        case 4096: return launch_update_L4096(mode, nf, a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ypass(int mode, int L, const YArgs& ya, const LaunchArgs& a) {
    switch (L) {
        case 8: return launch_ypass_L8(mode, ya, a);
        case 16: return launch_ypass_L16(mode, ya, a);
        case 32: return launch_ypass_L32(mode, ya, a);
        case 64: return launch_ypass_L64(mode, ya, a);
        case 128: return launch_ypass_L128(mode, ya, a);
        case 256: return launch_ypass_L256(mode, ya, a);
        case 512: return launch_ypass_L512(mode, ya, a);
        case 1024: return launch_ypass_L1024(mode, ya, a);
        case 2048: return launch_ypass_L2048(mode, ya, a);
        case 4096: return launch_ypass_L4096(mode, ya, a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_xrow(int mode, int L, int ng, const LaunchArgs& a) {
    switch (L) {
        case 8: return launch_xrow_L8(mode, ng, a);
        case 16: return launch_xrow_L16(mode, ng, a);
        case 32: return launch_xrow_L32(mode, ng, a);
        case 64: return launch_xrow_L64(mode, ng, a);
        case 128: return launch_xrow_L128(mode, ng, a);
        case 256: return launch_xrow_L256(mode, ng, a);
        case 512: return launch_xrow_L512(mode, ng, a);
        case 1024: return launch_xrow_L1024(mode, ng, a);
        case 2048: return launch_xrow_L2048(mode, ng, a);
        case 4096: return launch_xrow_L4096(mode, ng, a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjcol(int mode, int L, const AdjArgs& aa, const LaunchArgs& a) {
    switch (L) {
        case 8: return launch_adjcol_L8(mode, aa, a);
        case 16: return launch_adjcol_L16(mode, aa, a);
        case 32: return launch_adjcol_L32(mode, aa, a);
        case 64: return launch_adjcol_L64(mode, aa, a);
        case 128: return launch_adjcol_L128(mode, aa, a);
        case 256: return launch_adjcol_L256(mode, aa, a);
        case 512: return launch_adjcol_L512(mode, aa, a);
        case 1024: return launch_adjcol_L1024(mode, aa, a);
        case 2048: return launch_adjcol_L2048(mode, aa, a);
        case 4096: return launch_adjcol_L4096(mode, aa, a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjseed(hipStream_t s, const float2* phi, float2* g, const float* coef, int nshell, int nx, int ny,
                          int tc) {
    const int64_t total = static_cast<int64_t>(nx / 2) * ny;
    hipLaunchKernelGGL(adjseed_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, phi, g, coef,
                       nshell, nx, ny, tc);
    return hipGetLastError();
}

hipError_t launch_advance(hipStream_t s, uint64_t* step_ctr, int64_t k) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(64), 0, s, step_ctr, k);
    return hipGetLastError();
}

hipError_t launch_advance_many(hipStream_t s, uint64_t* const* ctrs, int n, int64_t k) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(advance_many_kernel, dim3((n + 255) / 256), dim3(256), 0, s, ctrs, n, k);
    return hipGetLastError();
}

hipError_t launch_apply_frame(hipStream_t s, float* real, const int2* frame, int n) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(apply_frame_kernel, dim3((n + 255) / 256), dim3(256), 0, s, real, frame, n);
    return hipGetLastError();
}

hipError_t launch_take_flags(hipStream_t s, uint64_t* const* ctrs, int n, uint32_t* out) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(take_flags_kernel, dim3((n + 255) / 256), dim3(256), 0, s, ctrs, n, out);
    return hipGetLastError();
}

hipError_t launch_init_uniform(hipStream_t s, float* out, int64_t n, uint32_t field, uint32_t key0, uint32_t key1,
                               double lo, double hi) {
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(init_uniform_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, out, n, field, key0,
                       key1, lo, hi);
    return hipGetLastError();
}

hipError_t launch_shells(hipStream_t s, const float2* S, int nx, int ny, int nz, int tc, int ndim, double scale,
                         int nshell, unsigned long long* acc) {
    if (nshell < 1) return hipSuccess;
    unsigned long long* hi = acc;
    unsigned long long* lo = acc + nshell;
    unsigned long long* cnt = acc + 2 * nshell;
    auto* key = reinterpret_cast<unsigned int*>(acc + 3 * nshell);
    hipLaunchKernelGGL(shell_keys_kernel, dim3(256), dim3(256), sizeof(unsigned int) * nshell, s, S, nx, ny, nz, tc,
                       ndim, scale, nshell, key);
    const size_t lds = nshell * (2 * sizeof(unsigned long long) + 2 * sizeof(unsigned int));
    hipLaunchKernelGGL(shell_sums_kernel, dim3(256), dim3(256), lds, s, S, nx, ny, nz, tc, ndim, scale, nshell, key,
                       hi, lo, cnt);
    hipLaunchKernelGGL(shell_means_kernel, dim3((nshell + 255) / 256), dim3(256), 0, s, nshell, key, hi, lo, cnt);
    return hipGetLastError();
}

hipError_t launch_philox(hipStream_t s, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                         int64_t count, uint32_t* out) {
    const int64_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(philox_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, c0, c1, c2, c3, k0, k1,
                       count, out);
    return hipGetLastError();
}

#endif  // PSS_COMMON

}  // namespace pss
