// kernels.hip -- HIP kernels of libtq for CDNA4 (gfx950), wave64.
//
// State vectors are complex64 (float2) rows of 2^n amplitudes in HBM.  Every
// sweep over a state is a tile kernel: a 256-thread workgroup stages tiles of
// 2^t amplitudes in LDS (t index bits = the `c` lowest bits, so that each
// wavefront reads contiguous runs, plus `h` high bits), works on them and
// writes them back.  Gate matrices are resolved from the symbol values and
// pre-multiplied (fused) in float64 by a separate builder kernel and rounded
// once to complex64.  All reductions are two-stage and fixed-order (no
// floating-point atomics), so every output is bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "device_ops.h"
#include "kernels.h"

namespace tq {

// ---------------------------------------------------- gate matrices (fp64)
// Closed forms of the opcode set, written from the gate definitions: for an
// involutory generator G, G^t = (1+w)/2 I + (1-w)/2 G with w = e^{i pi t}
// (the phase convention e^{i pi t/2}(cos(pi t/2) I - i sin(pi t/2) G)), and a
// rotation exp(-i theta G / 2) = cos(theta/2) I - i sin(theta/2) G.
//
// Gates whose matrix is a global phase times a matrix of simpler form are
// built without that phase: RZ(theta) = e^{-i theta/2} diag(1, e^{i theta}),
// RZZ(gamma) = e^{-i gamma/2} diag(1, e^{i gamma}, e^{i gamma}, 1) (entries
// exactly 1), X^t, sqrt X, XX^t, YY^t = e^{i pi t/2}(cos I - i sin G) (real
// diagonal, imaginary off-diagonal), Y^t, sqrt Y = e^{i pi t/2}(cos I - i sin
// Y) (real), sqrt W = e^{i pi/4}(cos(pi/4) I - i sin(pi/4) W) (real diagonal).  The phases of a row sum to one global phase, a linear form in
// the parameters that the planner lists per group (PhaseTerm), which the
// builder multiplies into the first qubit's product-init matrix:
// states and amplitudes come out with the gates' own phases, while every
// intermediate state differs from its phased counterpart by a global phase
// alone, which no expectation, gradient or probability sees.
//
// The table is callable from the host as well (gate_table_host), so that the
// matrices and derivatives the builder forms can be checked on the CPU.
struct cd {
    double x, y;
};
__host__ __device__ __forceinline__ cd C(double x, double y) { return cd{x, y}; }
__host__ __device__ __forceinline__ cd cdmul(cd a, cd b) { return cd{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__host__ __device__ __forceinline__ cd cdadd(cd a, cd b) { return cd{a.x + b.x, a.y + b.y}; }

// sin and cos of x, and of pi x
__host__ __device__ __forceinline__ void sc(double x, double *s, double *c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    sincos(x, s, c);
#else
    *s = std::sin(x);
    *c = std::cos(x);
#endif
}
__host__ __device__ __forceinline__ void scpi(double x, double *s, double *c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    sincospi(x, s, c);
#else
    *s = std::sin(M_PI * x);
    *c = std::cos(M_PI * x);
#endif
}

// m: row-major d x d, zero-initialised by the caller
__host__ __device__ __forceinline__ int gate_matrix_dev(int op, const double *eta, const double *ex, int form, cd *m)
{
    const double r = 0.70710678118654752440;
    double c, s;
    switch (op) {
    case OP_H: m[0] = C(r, 0); m[1] = C(r, 0); m[2] = C(r, 0); m[3] = C(-r, 0); return 2;
    case OP_X: m[1] = C(1, 0); m[2] = C(1, 0); return 2;
    case OP_Y: m[1] = C(0, -1); m[2] = C(0, 1); return 2;
    case OP_Z: m[0] = C(1, 0); m[3] = C(-1, 0); return 2;
    case OP_RX:
        sc(eta[0] * 0.5, &s, &c);
        m[0] = C(c, 0); m[1] = C(0, -s); m[2] = C(0, -s); m[3] = C(c, 0); return 2;
    case OP_RY:
        sc(eta[0] * 0.5, &s, &c);
        m[0] = C(c, 0); m[1] = C(-s, 0); m[2] = C(s, 0); m[3] = C(c, 0); return 2;
    case OP_RZ:
        sc(eta[0], &s, &c);
        m[0] = C(1, 0); m[3] = C(c, s); return 2;
    case OP_XPOW: case OP_SQRTX: case OP_YPOW: case OP_SQRTY: {
        scpi(0.5 * (op == OP_XPOW || op == OP_YPOW ? eta[0] : 0.5), &s, &c);
        m[0] = m[3] = C(c, 0);
        if (op == OP_XPOW || op == OP_SQRTX) { m[1] = m[2] = C(0, -s); }
        else { m[1] = C(-s, 0); m[2] = C(s, 0); }
        return 2;
    }
    case OP_ZPOW:
        scpi(eta[0], &s, &c);
        m[0] = C(1, 0); m[3] = C(c, s); return 2;
    case OP_SQRTW:
        // W^{1/2} = e^{i pi/4} (cos(pi/4) I - i sin(pi/4) W) with W = [[0, e^{-i pi/4}],
        // [e^{i pi/4}, 0]]: without the phase, r I - i r W with r = 1/sqrt(2)
        // (real diagonal; -i r e^{-/+ i pi/4} = (-1 -/+ i)/2 off it)
        m[0] = m[3] = C(r, 0); m[1] = C(-0.5, -0.5); m[2] = C(0.5, -0.5);
        return 2;
    case OP_CZ:
        m[0] = m[5] = m[10] = C(1, 0); m[15] = C(-1, 0); return 4;
    case OP_CZPOW:
        scpi(eta[0], &s, &c);
        m[0] = m[5] = m[10] = C(1, 0); m[15] = C(c, s); return 4;
    case OP_CNOT:
        if (form == FORM_CBLOCK) { m[1] = m[2] = C(1, 0); return 2; }
        m[0] = m[5] = C(1, 0); m[11] = m[14] = C(1, 0); return 4;
    case OP_CNOTPOW: {
        scpi(eta[0], &s, &c);
        cd a = C(0.5 * (1 + c), 0.5 * s), bq = C(0.5 * (1 - c), -0.5 * s);
        if (form == FORM_CBLOCK) { m[0] = m[3] = a; m[1] = m[2] = bq; return 2; }
        m[0] = m[5] = C(1, 0); m[10] = m[15] = a; m[11] = m[14] = bq; return 4;
    }
    case OP_XXPOW: {  // cos I - i sin XX; XX couples 00 with 11 and 01 with 10, all with +1
        scpi(0.5 * eta[0], &s, &c);
        m[0] = m[5] = m[10] = m[15] = C(c, 0);
        m[3] = m[6] = m[9] = m[12] = C(0, -s);
        return 4;
    }
    case OP_YYPOW: {  // cos I - i sin YY; YY = -|11><00| - |00><11| + |10><01| + |01><10|
        scpi(0.5 * eta[0], &s, &c);
        m[0] = m[5] = m[10] = m[15] = C(c, 0);
        m[3] = m[12] = C(0, s);
        m[6] = m[9] = C(0, -s);
        return 4;
    }
    case OP_ZZPOW:
        scpi(eta[0], &s, &c);
        m[0] = m[15] = C(1, 0); m[5] = m[10] = C(c, s); return 4;
    case OP_RZZ:
        sc(eta[0], &s, &c);
        m[0] = m[15] = C(1, 0); m[5] = m[10] = C(c, s); return 4;
    case OP_FSIM:
        sc(eta[0], &s, &c);
        m[0] = C(1, 0); m[5] = m[10] = C(c, 0); m[6] = m[9] = C(0, -s);
        sc(eta[1], &s, &c);
        m[15] = C(c, -s); return 4;
    case OP_SWAP:
        m[0] = m[6] = m[9] = m[15] = C(1, 0); return 4;
    case OP_MATRIX1:
        for (int i = 0; i < 4; i++) m[i] = C(ex[2 * i], ex[2 * i + 1]);
        return 2;
    case OP_MATRIX2:
        for (int i = 0; i < 16; i++) m[i] = C(ex[2 * i], ex[2 * i + 1]);
        return 4;
    }
    return 0;
}

// derivative of gate_matrix_dev (the matrix as built, without its left-out
// phase) with respect to parameter `which` (m zero-initialised)
__host__ __device__ __forceinline__ int gate_deriv_dev(int op, const double *eta, int which, int form, cd *m)
{
    double c, s;
    const double pi = 3.14159265358979323846;
    switch (op) {
    case OP_RX:
        sc(eta[0] * 0.5, &s, &c);
        m[0] = C(-0.5 * s, 0); m[1] = C(0, -0.5 * c); m[2] = C(0, -0.5 * c); m[3] = C(-0.5 * s, 0); return 2;
    case OP_RY:
        sc(eta[0] * 0.5, &s, &c);
        m[0] = C(-0.5 * s, 0); m[1] = C(-0.5 * c, 0); m[2] = C(0.5 * c, 0); m[3] = C(-0.5 * s, 0); return 2;
    case OP_RZ:  // d/dtheta diag(1, e^{i theta})
        sc(eta[0], &s, &c);
        m[3] = C(-s, c); return 2;
    case OP_RZZ:
        sc(eta[0], &s, &c);
        m[5] = m[10] = C(-s, c); return 4;
    case OP_XPOW: case OP_YPOW: case OP_XXPOW: case OP_YYPOW: {
        // d/dt (cos(pi t/2) I - i sin(pi t/2) G) = (pi/2)(-sin I - i cos G): the
        // diagonal ds, and -i dc times each entry of G.  Every entry is its own
        // expression (a negated copy of a complex value with a zero part has
        // been compiled for the device with the sign of only one part flipped).
        scpi(0.5 * eta[0], &s, &c);
        const double ds = -0.5 * pi * s, dc = 0.5 * pi * c;
        switch (op) {
        case OP_XPOW: m[0] = m[3] = C(ds, 0); m[1] = m[2] = C(0, -dc); return 2;
        case OP_YPOW: m[0] = m[3] = C(ds, 0); m[1] = C(-dc, 0); m[2] = C(dc, 0); return 2;
        case OP_XXPOW: m[0] = m[5] = m[10] = m[15] = C(ds, 0); m[3] = m[6] = m[9] = m[12] = C(0, -dc); return 4;
        default:  // YY: -1 on (00, 11) and (11, 00), +1 on (01, 10) and (10, 01)
            m[0] = m[5] = m[10] = m[15] = C(ds, 0); m[3] = m[12] = C(0, dc); m[6] = m[9] = C(0, -dc); return 4;
        }
    }
    case OP_ZPOW: case OP_CZPOW: case OP_CNOTPOW: case OP_ZZPOW: {
        // d/dt G^t = (i pi w / 2)(I - G), w = e^{i pi t}: i pi w / 2 = (kx, ky)
        scpi(eta[0], &s, &c);
        const double kx = -0.5 * pi * s, ky = 0.5 * pi * c;
        switch (op) {
        case OP_ZPOW: m[3] = C(2 * kx, 2 * ky); return 2;
        case OP_CZPOW: m[15] = C(2 * kx, 2 * ky); return 4;
        case OP_CNOTPOW:
            if (form == FORM_CBLOCK) { m[0] = m[3] = C(kx, ky); m[1] = m[2] = C(-kx, -ky); return 2; }
            m[10] = m[15] = C(kx, ky); m[11] = m[14] = C(-kx, -ky); return 4;
        default: m[5] = m[10] = C(2 * kx, 2 * ky); return 4;  // ZZPOW
        }
    }
    case OP_FSIM:
        if (which == 0) {
            sc(eta[0], &s, &c);
            m[5] = m[10] = C(-s, 0); m[6] = m[9] = C(0, -c);
        } else {
            sc(eta[1], &s, &c);
            m[15] = C(-s, -c);  // -i e^{-i phi}
        }
        return 4;
    }
    return 0;
}

int gate_table_host(int op, const double *eta, const double *ex, int form, int deriv, int which, double *out)
{
    cd m[16];
    for (int i = 0; i < 16; i++) m[i] = C(0, 0);
    const int d = deriv ? gate_deriv_dev(op, eta, which, form, m) : gate_matrix_dev(op, eta, ex, form, m);
    for (int i = 0; i < d * d; i++) {
        out[2 * i] = m[i].x;
        out[2 * i + 1] = m[i].y;
    }
    return d;
}

// permutation of a 4x4 two-qubit matrix for reversed qubit order (|ab> -> |ba>)
__host__ __device__ __forceinline__ void swap_qubits4(cd *m)
{
    cd t[16];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int pi = (i == 1) ? 2 : (i == 2) ? 1 : i, pj = (j == 1) ? 2 : (j == 2) ? 1 : j;
            t[pi * 4 + pj] = m[i * 4 + j];
        }
#pragma unroll
    for (int i = 0; i < 16; i++) m[i] = t[i];
}

// Where the builder finds one batch row's parameters.
struct BuildCtx {
    const Member *members;
    const GateDev *gates;
    const int32_t *slot_sym;
    const double *scale, *off;  // this row's scale and offset per slot
    const double *explicit_mats;
    const float *theta;         // this row's symbol values
    uint64_t noise_seed;        // channels: the row's trajectory draws
    int64_t b;                  // batch row
    const ShiftDev *shift;      // derived rows: the row's parameter moves (else NULL)
    double eps;                 // symbol moves are dtheta x eps
};

__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t counter);

// The Pauli (0 = I, 1 = X, 2 = Y, 3 = Z) a Pauli channel applies in batch row
// b, one trajectory of the noisy circuit (Sec. "Noise in qsim": one Kraus
// operator drawn per channel): r = (u >> 11) 2^-53 with u the output number
// (b 2^32 + k) of SplitMix64 from the noise seed, k the channel's ordinal in
// the circuit; X if r < p_x, Y if r < p_x + p_y, Z if r < p_x + p_y + p_z
// (fp64, in that order), else I.
__device__ __forceinline__ int channel_pick(uint64_t seed, int64_t b, int k, const double *p)
{
    const uint64_t u = splitmix64(seed, ((uint64_t)b << 32) | (uint64_t)(uint32_t)k);
    const double r = (double)(u >> 11) * 0x1.0p-53;
    if (r < p[0]) return 1;
    if (r < p[0] + p[1]) return 2;
    if (r < p[0] + p[1] + p[2]) return 3;
    return 0;
}

// symbol resolution eta = scale*theta + offset (or the constant) of a parameter slot
// (derived rows: the symbol value moved by dtheta, eta moved by delta)
__device__ __forceinline__ double slot_value(const BuildCtx &c, int slot)
{
    const int sy = c.slot_sym[slot];
    if (!c.shift) return sy >= 0 ? c.scale[slot] * (double)c.theta[sy] + c.off[slot] : c.off[slot];
    const ShiftDev &x = *c.shift;
    if (sy < 0) return c.off[slot];
    const double th = sy == x.sym ? (double)c.theta[sy] + x.dtheta * c.eps : (double)c.theta[sy];
    const double eta = c.scale[slot] * th + c.off[slot];
    return slot == x.slot[0] ? eta + x.delta[0] : slot == x.slot[1] ? eta + x.delta[1] : eta;
}
__device__ __forceinline__ void resolve(const BuildCtx &c, const GateDev &gd, double *eta)
{
    for (int j = 0; j < gd.np; j++) eta[j] = slot_value(c, gd.slot0 + j);
}

// Half turns of a forward rotation task: rint(phi / pi) of its angle phi (the
// sum over its members, all about one axis), the matrix being cos phi I - i
// sin phi G.
__device__ __forceinline__ int rot_turns(const BuildTask &bt, const BuildCtx &c)
{
    double phi = 0.0;  // in units of pi
    for (int mi = 0; mi < bt.mem_count; mi++) {
        const GateDev gd = c.gates[c.members[bt.mem_begin + mi].gate];
        const double eta = gd.np ? slot_value(c, gd.slot0) : 0.5;  // sqrt X, sqrt Y: G^(1/2)
        phi += gd.op == OP_RX || gd.op == OP_RY ? eta * (0.5 / 3.14159265358979323846) : 0.5 * eta;
    }
    return (int)((long long)rint(phi) & 1);
}

// Rotation [[c, -s], [s, c]] up to its sign as three shears: with c >= 0 it is
// [1 p; 0 1] [1 0; s 1] [1 p; 0 1], p = -s / (1 + c), |p| <= 1: three FMAs per
// pair and component, in place, where the matrix takes two multiplies and two
// FMAs into new registers (QAOA cost, 20 qubits x 256 rows: the VALU-bound
// passes 7.1 -> 6.7 ms per step; VQE forward passes, 16 qubits x 4096 rows,
// 16.8 -> 14.8 ms together with the X index maps).  A rotation with c < 0 is taken as minus the one by
// the angle less pi; `odd` says so (forward tasks: from the angle itself, so
// that the row's phase, which takes these signs up, counts the same ones).
__device__ __forceinline__ double2 shear_of(double c, double s, bool odd)
{
    if (odd) {
        c = -c;
        s = -s;
    }
    return make_double2(-s / (1.0 + c), s);
}

// One build task for one row: symbol resolution eta = scale*theta + offset
// and the fused product / dagger / derivative, all in float64.  D is the
// matrix dimension; fixed at compile time so every array stays in registers.
// Returns 1 when its shears leave out a sign that belongs to the row's phase.
template <int D> __device__ __forceinline__ int build_task_d(const BuildTask &bt, const BuildCtx &c, double2 *out)
{
    cd acc[16], g[16];
#pragma unroll
    for (int i = 0; i < 16; i++) acc[i] = C(0, 0);
#pragma unroll
    for (int i = 0; i < D; i++) acc[i * D + i] = C(1, 0);
    for (int mi = 0; mi < bt.mem_count; mi++) {
        const Member mem = c.members[bt.mem_begin + mi];
        const GateDev gd = c.gates[mem.gate];
        double eta[3] = {0, 0, 0};
        resolve(c, gd, eta);
        const double *ex = gd.explicit_ >= 0 ? c.explicit_mats + 32 * gd.explicit_ : nullptr;
#pragma unroll
        for (int i = 0; i < 16; i++) g[i] = C(0, 0);
        int gdim;
        if (gd.op == OP_PCHAN) {  // this row's Pauli (never a derivative: no symbols)
            const int k = channel_pick(c.noise_seed, c.b, gd.chan, eta);
            if (k == 0) { g[0] = g[3] = C(1, 0); }
            else if (k == 1) { g[1] = g[2] = C(1, 0); }
            else if (k == 2) { g[1] = C(0, -1); g[2] = C(0, 1); }
            else { g[0] = C(1, 0); g[3] = C(-1, 0); }
            gdim = 2;
        } else {
            gdim = bt.kind == BT_DERIV ? gate_deriv_dev(gd.op, eta, bt.which, mem.form, g)
                                       : gate_matrix_dev(gd.op, eta, ex, mem.form, g);
        }
        if (gdim != D) continue;  // the planner never mixes dimensions
        if (D == 4 && mem.swapped) swap_qubits4(g);
        if (bt.kind == BT_DAGGER) {
#pragma unroll
            for (int i = 0; i < D; i++)
#pragma unroll
                for (int j = 0; j < D; j++) acc[i * D + j] = C(g[j * D + i].x, -g[j * D + i].y);
        } else if (bt.kind == BT_DERIV || bt.mem_count == 1) {  // one member: its matrix itself
#pragma unroll
            for (int i = 0; i < D * D; i++) acc[i] = g[i];
        } else {
            cd t[16];
#pragma unroll
            for (int i = 0; i < D; i++)
#pragma unroll
                for (int j = 0; j < D; j++) {
                    cd sacc = C(0, 0);
#pragma unroll
                    for (int k = 0; k < D; k++) sacc = cdadd(sacc, cdmul(g[i * D + k], acc[k * D + j]));
                    t[i * D + j] = sacc;
                }
#pragma unroll
            for (int i = 0; i < D * D; i++) acc[i] = t[i];
        }
    }
    if (bt.diag == 4) {
        // excitation preserving: |00> phase, the (|01>, |10>) block, |11> phase
        const int ix[6] = {0, 5, 6, 9, 10, 15};
#pragma unroll
        for (int i = 0; i < 6; i++) out[i] = make_double2(acc[ix[i]].x, acc[ix[i]].y);
    } else if (bt.diag >= 2) {
        // a I + b P: a from entry (0,0), b from entry (0,3) (P_03 = 1 for XX, -1 for YY)
        const double sg = bt.diag == 3 ? -1.0 : 1.0;
        out[0] = make_double2(acc[0].x, acc[0].y);
        out[1] = make_double2(sg * acc[D - 1].x, sg * acc[D - 1].y);
    } else if (bt.diag) {
#pragma unroll
        for (int i = 0; i < D; i++) out[i] = make_double2(acc[i * D + i].x, acc[i * D + i].y);
    } else {
#pragma unroll
        for (int i = 0; i < D * D; i++) out[i] = make_double2(acc[i].x, acc[i].y);
    }
    if (bt.kind == BT_DERIV || bt.which == BX_NONE) return 0;
    const bool fwd = bt.kind == BT_PRODUCT;
    const double cr = acc[0].x, sr = D == 4 ? -out[1].y : bt.which == BX_REAL ? acc[D].x : -acc[D].y;
    const bool odd = fwd ? rot_turns(bt, c) != 0 : cr < 0.0;
    out[D == 4 ? 2 : 4] = shear_of(cr, sr, odd);
    return fwd && odd;
}

__device__ __forceinline__ int build_task(const BuildTask &bt, const BuildCtx &c, double2 *out)
{
    return bt.dim == 2 ? build_task_d<2>(bt, c, out) : build_task_d<4>(bt, c, out);
}

// --------------------------------------------------- matrix build kernel
// One thread per (row, task); the result goes to the row's matrix block.
template <class A>
__device__ __forceinline__ void build_rows(const A &a, const float *theta, uint64_t noise_seed, int row, int bx)
{
    const int ti = bx * blockDim.x + threadIdx.x + a.task_begin;
    // derived rows take the symbols, parameter tables and trajectory of
    // their source row, plus their parameter moves
    int src = row;
    const ShiftDev *shift = nullptr;
    if (a.x_period > 0) {
        const int64_t L = a.x_begin + row;
        src = (int)(L / a.x_period);
        shift = a.x_shift + (L - (int64_t)src * a.x_period);
    }
    const int b = cget(a.rows, src);
    BuildCtx c{a.members, a.gates, a.slot_sym,
               a.slot_scale + (a.uniform ? 0 : (int64_t)src * a.n_slots),
               a.slot_off + (a.uniform ? 0 : (int64_t)src * a.n_slots), a.explicit_mats,
               theta + (int64_t)b * a.S, noise_seed, b, shift, a.x_eps};
    int odd = 0;
    if (ti < a.task_end) {
        const BuildTask bt = a.tasks[ti];
        odd = build_task(bt, c, a.mats + (int64_t)row * a.mat_stride + bt.out);
    }
    if (a.phase_out < 0 || bx != 0) return;
    // the row's global phase (block 0 of the row; its thread 0 built the
    // product-init matrix at phase_out), reduced in a fixed order
    __shared__ double part[4];
    // (signs the shears of forward rotations leave out: this block's tasks,
    // then the tasks of the row's other blocks)
    for (int j = ti + blockDim.x; j < a.rot_end; j += blockDim.x) {
        const BuildTask bt = a.tasks[j];
        if (bt.kind == BT_PRODUCT && bt.which != BX_NONE) odd += rot_turns(bt, c);
    }
    double ph = odd * 3.14159265358979323846;
    for (int j = threadIdx.x; j < a.n_phase; j += blockDim.x) {
        const PhaseTerm pt = a.phase_terms[j];
        ph += pt.slot >= 0 ? pt.c * slot_value(c, pt.slot) : pt.c;
    }
    ph = wave_sum(ph);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ph;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s, co;
        sc(part[0] + part[1] + part[2] + part[3], &s, &co);
        double2 *out = a.mats + (int64_t)row * a.mat_stride + a.phase_out;
        for (int i = 0; i < 4; i++) {
            const double2 v = out[i];
            out[i] = make_double2(co * v.x - s * v.y, co * v.y + s * v.x);
        }
    }
}

__global__ __launch_bounds__(256) void k_build_mats(BuildArgs a)
{
    build_rows(a, a.theta, a.noise_seed, blockIdx.y, blockIdx.x);
}

// Derived rows of the batched shift rules, one wavefront per row (four rows
// per workgroup): the source row's matrices (x_copy entries of its block)
// copied into the derived row's block ...
__global__ __launch_bounds__(256) void k_copy_source(BuildArgs a, int nrows)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= nrows) return;
    const int64_t L = a.x_begin + row;
    const int src = (int)(L / a.x_period);
    const double2 *from = a.x_src + (int64_t)src * a.mat_stride;
    double2 *to = a.mats + (int64_t)row * a.mat_stride;
    for (int e = lane; e < a.x_copy; e += 64) to[e] = from[e];
}

// ... then the tasks that read a moved parameter built again, one thread per
// row (a move's list holds a task or two); the row's global phase, as in
// k_build_mats, multiplied into the product-init task when it heads the
// list, else the change of the moved parameters' phase terms multiplied into
// the copied product-init matrix.  (The signs of the rotations' shears are
// left out: derived rows only give expectations.)
__global__ __launch_bounds__(256) void k_build_list(BuildArgs a, int nrows)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= nrows) return;
    const int64_t L = a.x_begin + row;
    const int src = (int)(L / a.x_period);
    const int m = (int)(L - (int64_t)src * a.x_period);
    const ShiftDev *shift = a.x_shift + m;
    const int b = cget(a.rows, src);
    BuildCtx c{a.members, a.gates, a.slot_sym,
               a.slot_scale + (a.uniform ? 0 : (int64_t)src * a.n_slots),
               a.slot_off + (a.uniform ? 0 : (int64_t)src * a.n_slots), a.explicit_mats,
               a.theta + (int64_t)b * a.S, a.noise_seed, b, shift, a.x_eps};
    double2 *block = a.mats + (int64_t)row * a.mat_stride;
    for (int li = a.list_begin[m]; li < a.list_begin[m + 1]; li++) {
        const BuildTask bt = a.tasks[a.task_list[li]];
        build_task(bt, c, block + bt.out);
    }
    if (a.phase_out < 0) return;
    double ph = 0.0;
    if (a.phase_full[m]) {
        for (int j = 0; j < a.n_phase; j++) {
            const PhaseTerm pt = a.phase_terms[j];
            ph += pt.slot >= 0 ? pt.c * slot_value(c, pt.slot) : pt.c;
        }
    } else {
        if (a.phase_begin[m] == a.phase_begin[m + 1]) return;
        BuildCtx c0 = c;
        c0.shift = nullptr;
        for (int j = a.phase_begin[m]; j < a.phase_begin[m + 1]; j++) {
            const PhaseTerm pt = a.phase_terms[a.phase_list[j]];
            ph += pt.c * (slot_value(c, pt.slot) - slot_value(c0, pt.slot));
        }
    }
    double sn, co;
    sc(ph, &sn, &co);
    double2 *out = block + a.phase_out;
    for (int i = 0; i < 4; i++) {
        const double2 v = out[i];
        out[i] = make_double2(co * v.x - sn * v.y, co * v.y + sn * v.x);
    }
}

template <class A> __device__ __forceinline__ void build_stage(const A &a, int row, int si)
{
    const int j = threadIdx.x;
    const Stage st = cget(a.stages, cget(a.list, si));
    if (j >= (1 << st.r)) return;
    double2 *block = a.mats + (int64_t)row * a.mat_stride;
    double2 *out = block + st.mat;
    switch (st.r) {
    case 4:
        if constexpr (kStageBitsFwd >= 4) build_stage_r<4>(st, a.ops, block, out, j);
        break;
    case 3: build_stage_r<3>(st, a.ops, block, out, j); break;
    case 2: build_stage_r<2>(st, a.ops, block, out, j); break;
    default: build_stage_r<1>(st, a.ops, block, out, j); break;
    }
}
__global__ __launch_bounds__(64) void k_build_stage(StageBuildArgs a) { build_stage(a, blockIdx.y, blockIdx.x); }

// ------------------------------------------------------- forward pass
template <class A> __device__ __forceinline__ void run_pass(const A &a, float2 *state, int bid, unsigned char *smem)
{
    const PassCtx c = pass_setup(a, state, bid, smem);
    const SMat G = smat(a.mats + (int64_t)c.row * a.mat_stride);
    const int64_t ntiles = (int64_t)1 << a.tiles_log2;
    for (int64_t tile = c.w; tile < ntiles; tile += a.wg_per_row) {
        const uint64_t fb = pdep64((uint64_t)tile, a.g.fixed_mask);
        pass_load(a, c, fb);
        __syncthreads();
        for (int si = 0; si < a.nstages; si++) {
            const Stage st = cget(a.stages, si);
            run_stage_any(st, a.ops, c.lm, a.mat_begin, G, c.lds, a.g.t, fb, threadIdx.x, blockDim.x);
            __syncthreads();
        }
        pass_store(a, c, fb);
        __syncthreads();
    }
}
__global__ __launch_bounds__(256) void k_pass(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    run_pass(a, a.state, blockIdx.x, smem);
}

// ------------------------------------------------ Pauli sums on tiles
// The hardware hands consecutive workgroup ids to the 8 XCDs in turn; this
// renumbering gives each XCD a contiguous range of (row, tile) work so that
// the tiles of one row, which read each other as partner tiles, share that
// XCD's L2.
__device__ __forceinline__ int xcd_block(int bid, int nb)
{
    if (nb % 8) return bid;
    return (bid % 8) * (nb / 8) + bid / 8;
}

// Expectations of Pauli sums, and optionally phi = sum_k g_k h_k psi, over
// tiles of T = 256 P amplitudes (T < 256 when P == 1: the state is smaller).
// Thread tid owns the amplitudes l = tid + 256 r of the tile.  For each x
// group the thread forms d(l) = sum_t c'_t chi_{z_t}(l) from the group's
// terms (one sign per term and thread, one per u sub-group and register),
// reads the partner amplitudes psi_{l ^ x} once, and adds
// Re(conj(psi_l) d(l) psi_{l ^ x}) to the group's observable and
// g_k d(l) psi_{l ^ x} to phi_l.  Accumulation is in fp64; each workgroup
// reduces its expectation partials in a fixed order.
// bid, nb: the workgroup's number and the workgroups of the launch (or of its
// argument block); upstream: the call's gradients
template <int P, bool kPhi, class A>
__device__ __forceinline__ void run_pauli(const A &a, const float *upstream, int bid0, int nb, unsigned char *smem)
{
    const auto &g = a.g;
    const int T = 1 << g.t;
    float2 *la = reinterpret_cast<float2 *>(smem);
    uint64_t *hi_off = reinterpret_cast<uint64_t *>(la + T);
    double *red = reinterpret_cast<double *>(hi_off + (1 << g.h));  // [kPauliChunk][4 waves]
    double *esum = red + 4 * kPauliChunk;                           // [k_count]
    float2 *lb = reinterpret_cast<float2 *>(esum + a.k_count);      // partner tile (when any xF != 0)

    const int bid = xcd_block(bid0, nb);
    const int row = bid / a.wg_per_row, w = bid % a.wg_per_row;
    const int b = cget(a.rows, row);
    const float2 *ps = as_global(a.psi) + (int64_t)b * a.row_stride;
    const PChunk *chunks = a.chunks + cget(a.row_chunk_begin, row);
    const int nchunks = cget(a.row_chunk_count, row);
    const float *up = kPhi ? upstream + (int64_t)a.brows[row] * a.K : nullptr;
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const bool active = tid < T;
    const int kend = a.k_begin + a.k_count;
    build_hi_off(g, hi_off);
    for (int j = tid; j < a.k_count; j += blockDim.x) esum[j] = 0;
    TileCtx tc{hi_off, (1u << g.c) - 1, g.c};
    __syncthreads();

    const int64_t ntiles = (int64_t)1 << a.tiles_log2;
    for (int64_t tile = w; tile < ntiles; tile += a.wg_per_row) {
        const uint64_t fb = pdep64((uint64_t)tile, g.fixed_mask);
        tile_copy<true, (P > 1 ? P / 2 : 1)>(tc, la, const_cast<float2 *>(ps), fb, T);
        __syncthreads();
        float2 own[P];
#pragma unroll
        for (int r = 0; r < P; r++) own[r] = active ? la[sw(tid + 256 * r)] : make_float2(0.f, 0.f);
        double2 acc[kPhi ? P : 1];
#pragma unroll
        for (int r = 0; r < (kPhi ? P : 1); r++) acc[r] = make_double2(0.0, 0.0);

        for (int ci = 0; ci < nchunks; ci++) {
            const PChunk ch = cget(chunks, ci);
            if (ch.k0 < a.k_begin || ch.k0 >= kend) continue;
            double ek[kPauliChunk];
#pragma unroll
            for (int j = 0; j < kPauliChunk; j++) ek[j] = 0.0;
            for (int xi = ch.xf_begin; xi < ch.xf_end; xi++) {
                const PXfGroup xf = cget(a.xfg, xi);
                const float2 *src = la;
                if (xf.xF) {
                    __syncthreads();  // the previous partner tile is consumed
                    tile_copy<true, (P > 1 ? P / 2 : 1)>(tc, lb, const_cast<float2 *>(ps), fb ^ xf.xF, T);
                    __syncthreads();
                    src = lb;
                }
                for (int gi = xf.x_begin; gi < xf.x_end; gi++) {
                    const PXGroup xg = cget(a.xg, gi);
                    double dr[P], di[P];
#pragma unroll
                    for (int r = 0; r < P; r++) dr[r] = di[r] = 0.0;
                    for (int ui = xg.u_begin; ui < xg.u_end; ui++) {
                        const PUSub us = cget(a.us, ui);
                        double er = 0.0, ei = 0.0;
                        for (int ti = us.t_begin; ti < us.t_end; ti++) {
                            const PTerm tm = cget(a.terms, ti);
                            const double c = (par64(fb & tm.zF) ^ par32((uint32_t)tid & tm.zlo)) ? -tm.c : tm.c;
                            if (tm.im) ei += c;
                            else er += c;
                        }
#pragma unroll
                        for (int r = 0; r < P; r++) {
                            const double sg = (__popc(us.u & (uint32_t)r) & 1) ? -1.0 : 1.0;
                            dr[r] = fma(sg, er, dr[r]);
                            di[r] = fma(sg, ei, di[r]);
                        }
                    }
                    const bool self = xf.xF == 0 && xg.xT == 0;
                    const double gk = kPhi ? (double)up[ch.k0 + xg.kk] : 0.0;
                    double ex = 0.0;
                    if (!(xg.flags & 2)) {
#pragma unroll
                        for (int r = 0; r < P; r++) {
                            float2 pv = own[r];
                            if (!self && active) pv = src[sw((tid + 256 * r) ^ xg.xT)];
                            const double tr = dr[r] * (double)pv.x, ti = dr[r] * (double)pv.y;
                            ex = fma((double)own[r].x, tr, fma((double)own[r].y, ti, ex));
                            if (kPhi) {
                                acc[r].x = fma(gk, tr, acc[r].x);
                                acc[r].y = fma(gk, ti, acc[r].y);
                            }
                        }
                    } else {
#pragma unroll
                        for (int r = 0; r < P; r++) {
                            float2 pv = own[r];
                            if (!self && active) pv = src[sw((tid + 256 * r) ^ xg.xT)];
                            const double px = pv.x, py = pv.y;
                            const double tr = fma(dr[r], px, -di[r] * py), ti = fma(dr[r], py, di[r] * px);
                            ex = fma((double)own[r].x, tr, fma((double)own[r].y, ti, ex));
                            if (kPhi) {
                                acc[r].x = fma(gk, tr, acc[r].x);
                                acc[r].y = fma(gk, ti, acc[r].y);
                            }
                        }
                    }
#pragma unroll
                    for (int j = 0; j < kPauliChunk; j++) ek[j] += (j == xg.kk) ? ex : 0.0;
                }
            }
            // this tile's share of the chunk's expectations, in a fixed order
#pragma unroll
            for (int j = 0; j < kPauliChunk; j++)
                if (j < ch.nk) {
                    const double v = wave_sum(ek[j]);
                    if (lane == 0) red[j * 4 + wave] = v;
                }
            __syncthreads();
            if (tid < ch.nk)
                esum[ch.k0 - a.k_begin + tid] += ((red[tid * 4] + red[tid * 4 + 1]) + red[tid * 4 + 2]) + red[tid * 4 + 3];
            __syncthreads();
        }
        if (kPhi && active) {
            float2 *ph = as_global(a.phi) + (int64_t)b * a.row_stride;
#pragma unroll
            for (int r = 0; r < P; r++) {
                const uint64_t i = tile_index(tc, fb, tid + 256 * r);
                double2 v = acc[r];
                if (a.phi_accumulate) v = zadd(v, up2(ph[i]));
                ph[i] = down2(v);
            }
        }
        __syncthreads();
    }
    double *out = a.partial + ((int64_t)row * a.wg_per_row + w) * a.k_count;
    for (int j = tid; j < a.k_count; j += blockDim.x) out[j] = esum[j];
}
template <int P, bool kPhi> __global__ __launch_bounds__(256) void k_pauli(PauliArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    run_pauli<P, kPhi>(a, a.upstream, blockIdx.x, gridDim.x, smem);
}

// out[b, k] = sum over the row's workgroups of their partials: one block per
// (row, observable), strided sums then a tree, all in a fixed order.
template <class A> __device__ __forceinline__ void pauli_reduce(const A &a, float *dst, int row, int j)
{
    __shared__ double red[256];
    const double *p = a.partial + (int64_t)row * a.wg_per_row * a.k_count + j;
    double s = 0;
    for (int w = threadIdx.x; w < a.wg_per_row; w += blockDim.x) s += p[(int64_t)w * a.k_count];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) dst[(int64_t)a.rows[row] * a.K + a.k_begin + j] = (float)red[0];
}
__global__ __launch_bounds__(256) void k_pauli_reduce(PauliReduceArgs a)
{
    pauli_reduce(a, a.out, blockIdx.x, blockIdx.y);
}

// ------------------------------------------ diagonal Pauli sums in HBM
// Expectations of Z-only Pauli sums, streamed from HBM without LDS staging:
// workgroup w of a row sweeps the blocks w, w + wg_per_row, ... of the row,
// loading each thread's 16 amplitudes of the next block while it transforms
// the current one.  The class weights D(blk) are staged in LDS for
// kDiagRefill blocks at a time (a wave per class, a lane per block; classes
// past the chunk's get weight zero, so every block runs the same straight-line
// code).  Class c
// accumulates D(blk) W_v in its own register; the thread's sign chi_zT(tid)
// is applied once at the end, before the fixed-order reduction of each
// observable.
template <int A>
__global__ __launch_bounds__(256) void k_pauli_diag(DiagArgs a)
{
    __shared__ double dw[A * kDiagRefill];
    __shared__ double red[4];
    extern __shared__ __align__(16) unsigned char smem[];
    double *esum = reinterpret_cast<double *>(smem);  // [k_count]

    const int bid = xcd_block(blockIdx.x, gridDim.x);
    const int row = bid / a.wg_per_row, w = bid % a.wg_per_row;
    const int b = cget(a.rows, row);
    const float4 *ps = reinterpret_cast<const float4 *>(a.psi + (int64_t)b * a.row_stride);
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    // blocks of this workgroup: w + i wg_per_row for i < mine (w < wg_per_row <= blocks)
    const int64_t mine = (((int64_t)1 << a.blocks_log2) - w + a.wg_per_row - 1) / a.wg_per_row;
    const int kend = a.k_begin + a.k_count;
    const DChunk *chunks = a.chunks + cget(a.row_chunk_begin, row);
    const int nchunks = cget(a.row_chunk_count, row);
    for (int j = tid; j < a.k_count; j += blockDim.x) esum[j] = 0;

    for (int ci = 0; ci < nchunks; ci++) {
        const DChunk ch = cget(chunks, ci);
        if (ch.k_hi < a.k_begin || ch.k_lo >= kend) continue;
        const DClass *cls = a.classes + ch.c_begin;
        const int ncls = ch.c_end - ch.c_begin;
        double G[A];
        uint32_t vv[A];
#pragma unroll
        for (int c = 0; c < A; c++) {
            G[c] = 0.0;
            vv[c] = c < ncls ? cget(cls, c).v : 0u;
        }
        float4 nx[8];
        auto load = [&](int64_t i) {
            const float4 *src = ps + ((w + i * a.wg_per_row) << (kDiagBlockBits - 1)) + tid;
#pragma unroll
            for (int j = 0; j < 8; j++) nx[j] = src[256 * j];
        };
        load(0);
        for (int64_t i = 0; i < mine; i++) {
            const int slot = (int)(i % kDiagRefill);
            if (slot == 0) {
                __syncthreads();  // the previous weights are consumed
                const uint64_t blk = (uint64_t)(w + (i + lane) * a.wg_per_row);
                for (int c = wave; c < A; c += 4) {
                    double d = 0.0;  // classes past the chunk's weigh nothing
                    if (c < ncls) {
                        const DClass cc = cget(cls, c);
                        for (int t = cc.t_begin; t < cc.t_end; t++) {
                            const DTerm tm = cget(a.terms, t);
                            d += par64(blk & tm.zB) ? -tm.c : tm.c;
                        }
                    }
                    dw[lane * A + c] = d;
                }
                __syncthreads();
            }
            double p[16];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                p[2 * j] = fma((double)nx[j].x, (double)nx[j].x, (double)nx[j].y * (double)nx[j].y);
                p[2 * j + 1] = fma((double)nx[j].z, (double)nx[j].z, (double)nx[j].w * (double)nx[j].w);
            }
            if (i + 1 < mine) load(i + 1);
            // Walsh transform over the four register bits: p[v] = W_v
#pragma unroll
            for (int sb = 1; sb < 16; sb <<= 1)
#pragma unroll
                for (int r = 0; r < 16; r++)
                    if (!(r & sb)) {
                        const double x = p[r], y = p[r | sb];
                        p[r] = x + y;
                        p[r | sb] = x - y;
                    }
            double dv[A];
#pragma unroll
            for (int c = 0; c < A; c++) dv[c] = dw[slot * A + c];
#pragma unroll
            for (int c = 0; c < A; c++) G[c] = fma(dv[c], p[vv[c]], G[c]);
        }
        // thread signs, then one fixed-order reduction per observable
        const int k_first = ch.k_lo > a.k_begin ? ch.k_lo : a.k_begin;
        const int k_last = ch.k_hi < kend - 1 ? ch.k_hi : kend - 1;
        for (int k = k_first; k <= k_last; k++) {
            double e = 0.0;
#pragma unroll
            for (int c = 0; c < A; c++)
                if (c < ncls) {
                    const DClass cc = cget(cls, c);
                    if (cc.k == k) e += par32((uint32_t)tid & cc.zT) ? -G[c] : G[c];
                }
            const double v = wave_sum(e);
            if (lane == 0) red[wave] = v;
            __syncthreads();
            if (tid == 0) esum[k - a.k_begin] += ((red[0] + red[1]) + red[2]) + red[3];
            __syncthreads();
        }
    }
    __syncthreads();
    double *out = a.partial + ((int64_t)row * a.wg_per_row + w) * a.k_count;
    for (int j = tid; j < a.k_count; j += blockDim.x) out[j] = esum[j];
}

// ------------------------------------------------------ reverse pass
// psi and phi tiles side by side in LDS; the pass's matrices too.
template <class A> __device__ __forceinline__ void run_rev_pass(const A &a, int bid, unsigned char *smem)
{
    const RevCtx c = rev_setup(a, bid, smem);
    const int64_t ntiles = (int64_t)1 << a.tiles_log2;
    for (int64_t tile = c.w; tile < ntiles; tile += a.wg_per_row) {
        const uint64_t fb = pdep64((uint64_t)tile, a.g.fixed_mask);
        rev_load(a, c, fb);
        __syncthreads();
        for (int si = 0; si < a.nstages; si++) {
            const Stage st = cget(a.stages, si);
            run_rev_stage_any<kStageBitsRev>(st, a.ops, c.lm, a.mat_begin, c.lp, c.lf, a.g.t, fb, c.acc, a.gcount,
                                             a.gbase, threadIdx.x, blockDim.x);
            __syncthreads();
        }
        rev_store(a, c, fb);
        __syncthreads();
    }
    rev_finish(a, c);
}
__global__ __launch_bounds__(256, 2) void k_rev_pass(RevArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    run_rev_pass(a, blockIdx.x, smem);
}

// grad[b, s] = sum over gradient slots of s: 2 * scale * sum_w gpart
template <class A> __device__ __forceinline__ void grad_reduce(const A &a, float *grad, int row)
{
    const int b = cget(a.rows, row);
    const double *scale = a.slot_scale + (a.uniform ? 0 : (int64_t)row * a.n_slots);
    const double *p = a.gpart + (int64_t)row * a.wg_per_row * a.n_gslots;
    for (int s = threadIdx.x; s < a.S; s += blockDim.x) {
        double sum = 0;
        for (int k = a.sym_begin[s]; k < a.sym_begin[s + 1]; k++) {
            int gs = a.sym_gslots[k];
            double v = 0;
            for (int w = 0; w < a.wg_per_row; w++) v += p[(int64_t)w * a.n_gslots + gs];
            sum += 2.0 * scale[a.gslot_slot[gs]] * v;
        }
        grad[(int64_t)b * a.S + s] = (float)sum;
    }
}
__global__ void k_grad_reduce(GradReduceArgs a) { grad_reduce(a, a.grad, blockIdx.x); }

// ---------------------------------------------------- resident circuits
// Small circuits (psi, phi and every matrix of the row fit in LDS): one
// workgroup per batch row does the whole call -- product-state init, forward
// gates, expectations, H_g, reverse sweep, gradient reduction -- in one
// launch, on the matrices k_build_mats wrote.  At most 128 registers per
// thread, so that four rows share a CU.  Outputs are reduced in a fixed order.
template <class A, class C>
__device__ __forceinline__ void run_resident(const A &a, const C &c, int row, unsigned char *smem)
{
    const uint32_t T = 1u << a.n;
    const int tid = threadIdx.x, nt = blockDim.x;
    double *acc = reinterpret_cast<double *>(smem);                    // [waves][nacc]
    float2 *lp = reinterpret_cast<float2 *>(acc + (nt / 64) * a.nacc);  // [T]
    float2 *lf = lp + T;                                               // [T] (adjoint)
    const SMat M = smat(a.mats + (int64_t)row * a.mat_stride);
    resident_begin(a, M, acc, lp, tid, nt);
    for (int si = 0; si < a.nfstages; si++) {
        const Stage st = cget(a.fstages, si);
        run_stage_any(st, a.fops, M, 0, M, lp, a.n, 0, tid, nt);
        __syncthreads();
    }
    resident_middle(a, c, acc, lp, lf, row, tid, nt);
    if (c.grad)
        for (int si = 0; si < a.nrstages; si++) {
            const Stage st = cget(a.rstages, si);
            run_rev_stage_any<kStageBitsRevResident>(st, a.rops, M, 0, lp, lf, a.n, 0, acc, a.nacc, -a.gacc, tid, nt);
            __syncthreads();
        }
    resident_end(a, c, acc, row, tid, nt);
}
__global__ __launch_bounds__(256, 4) void k_resident(ResArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    run_resident(a, a, blockIdx.x, smem);
}

// ------------------------------------------------- merged launches
// A batch of many circuit structures (the paper's ops take any batch of
// circuits) would launch every step once per structure, each launch a row or
// two wide.  The same step of all structures is one launch instead: the
// workgroup takes its structure's argument block from a table that is read
// through the scalar cache, and the call's own pointers from `c`.  45
// structures of 2..13 qubits, adjoint: 5.7 ms as 140 launches, 0.41 ms as 11
// (the resident circuits 149 us, bound by the largest one's chain of stages).
template <class T> using TableArg = const __attribute__((address_space(4))) T;
template <class T> __device__ __forceinline__ TableArg<T> &table_arg(const void *table, int i)
{
    return reinterpret_cast<TableArg<T> *>(reinterpret_cast<uintptr_t>(table))[i];
}

__global__ __launch_bounds__(256) void k_build_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    const BatchBlock bb = cget(blocks, blockIdx.x);
    TableArg<BuildArgs> &a = table_arg<BuildArgs>(table, bb.arg);
    const int nx = (a.task_end - a.task_begin + 255) / 256;
    build_rows(a, c.theta, c.noise_seed, bb.block / nx, bb.block % nx);
}
__global__ __launch_bounds__(64) void k_stage_batch(const void *table, const BatchBlock *blocks, ResCall)
{
    const BatchBlock bb = cget(blocks, blockIdx.x);
    TableArg<StageBuildArgs> &a = table_arg<StageBuildArgs>(table, bb.arg);
    build_stage(a, bb.block / a.nlist, bb.block % a.nlist);
}
template <int NT>
__global__ __launch_bounds__(NT, 4) void k_resident_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const BatchBlock bb = cget(blocks, blockIdx.x);
    run_resident(table_arg<ResArgs>(table, bb.arg), c, bb.block, smem);
}
__global__ __launch_bounds__(256) void k_pass_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const BatchBlock bb = cget(blocks, blockIdx.x);
    TableArg<PassArgs> &a = table_arg<PassArgs>(table, bb.arg);
    run_pass(a, c.state_out ? c.state_out : a.state, bb.block, smem);
}
template <int P, bool kPhi>
__global__ __launch_bounds__(256) void k_pauli_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const BatchBlock bb = cget(blocks, blockIdx.x);
    // (1: the workgroup keeps its number; a structure's tiles share an XCD's
    // L2 only by chance, its few rows fit any)
    run_pauli<P, kPhi>(table_arg<PauliArgs>(table, bb.arg), c.upstream, bb.block, 1, smem);
}
__global__ __launch_bounds__(256) void k_pauli_reduce_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    const BatchBlock bb = cget(blocks, blockIdx.x);
    TableArg<PauliReduceArgs> &a = table_arg<PauliReduceArgs>(table, bb.arg);
    pauli_reduce(a, c.exp_out, bb.block / a.k_count, bb.block % a.k_count);
}
__global__ __launch_bounds__(256, 2) void k_rev_batch(const void *table, const BatchBlock *blocks, ResCall)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const BatchBlock bb = cget(blocks, blockIdx.x);
    run_rev_pass(table_arg<RevArgs>(table, bb.arg), bb.block, smem);
}
__global__ void k_grad_reduce_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    const BatchBlock bb = cget(blocks, blockIdx.x);
    grad_reduce(table_arg<GradReduceArgs>(table, bb.arg), c.grad, bb.block);
}

// ------------------------------------------------------------- sampling
__device__ __forceinline__ uint64_t weight_of(float2 v)
{
    double re = v.x, im = v.y;
    double p = re * re + im * im;
    return (uint64_t)(p * 0x1p62);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Level 1: the sum of the weights of each group of 64 amplitudes, streamed
// from HBM.  Eight consecutive lanes share a group: lane j of it sums the
// weights of amplitudes 8j .. 8j+7, read with four 16-byte loads when the row
// is 16-byte aligned (vec16), and the eight partial sums are added over the
// lanes.  Grid-stride over the groups of the row (integer sums: the order
// does not matter).
__global__ __launch_bounds__(256) void k_samp_l1(SampArgs a)
{
    const int row = blockIdx.y;
    const int sr = a.rows ? a.rows[row] : row;
    const float2 *st = a.state + (int64_t)sr * a.row_stride;
    uint64_t *out = a.levels + (int64_t)row * a.row_level + a.off[1];
    const int64_t N = a.count[0], ngrp = a.count[1];
    const int sub = threadIdx.x & 7;
    const int64_t stride = ((int64_t)gridDim.x * blockDim.x) >> 3;
    for (int64_t grp = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3; grp < ngrp; grp += stride) {
        const int64_t i0 = grp * 64 + sub * 8;
        uint64_t w = 0;
        if (a.vec16 && i0 + 8 <= N) {
            const float4 *p = reinterpret_cast<const float4 *>(st + i0);
            float4 v[4];
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] = p[k];
#pragma unroll
            for (int k = 0; k < 4; k++) w += weight_of(make_float2(v[k].x, v[k].y)) + weight_of(make_float2(v[k].z, v[k].w));
        } else {
            for (int e = 0; e < 8; e++)
                if (i0 + e < N) w += weight_of(st[i0 + e]);
        }
        // the eight lanes of a group are consecutive and take the same trip
        // count, so they are active together here
        w += __shfl_xor(w, 1, 8);
        w += __shfl_xor(w, 2, 8);
        w += __shfl_xor(w, 4, 8);
        if (sub == 0) out[grp] = w;
    }
}

// level k+1 from level k
__global__ __launch_bounds__(256) void k_samp_up(SampArgs a, int k)
{
    const int row = blockIdx.y;
    const int64_t grp = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    if (grp >= a.count[k + 1]) return;
    const int64_t i = grp * 64 + lane;
    const uint64_t *lv = a.levels + (int64_t)row * a.row_level;
    uint64_t wv = i < a.count[k] ? lv[a.off[k] + i] : 0;
    wv = wave_sum_u64(wv);
    if (lane == 0) a.levels[(int64_t)row * a.row_level + a.off[k + 1] + grp] = wv;
}

// SplitMix64 (Steele, Lea, Flood 2014): output number `counter` of the stream
// whose state starts at `seed`
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t counter)
{
    uint64_t z = seed + (counter + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// one wavefront per shot: descend the levels, at each one locating the child
// whose cumulative interval contains r by a wavefront prefix scan
__global__ __launch_bounds__(256) void k_samp_shots(SampArgs a)
{
    const int row = blockIdx.y;
    const int sr = a.rows ? a.rows[row] : row;
    const int b = a.brows ? a.brows[row] : row;
    const int64_t shot = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    if (shot >= a.n_shots) return;
    const uint64_t *lv = a.levels + (int64_t)row * a.row_level;
    const float2 *st = a.state + (int64_t)sr * a.row_stride;
    const int top = a.nlev;
    auto level_value = [&](int k, int64_t i) -> uint64_t {
        if (i >= a.count[k]) return 0;
        return k == 0 ? weight_of(st[i]) : lv[a.off[k] + i];
    };
    // total weight from the top level (at most 64 entries)
    const uint64_t tv = level_value(top, lane);
    const uint64_t W = wave_sum_u64(tv);
    uint64_t *out = a.out + (int64_t)b * a.n_shots + shot;
    if (W == 0) {
        // no distribution to draw from (an all-zero row): every shot is the
        // marker 2^64 - 1, which no bitstring of at most 32 qubits equals
        if (lane == 0) *out = ~0ull;
        return;
    }
    const uint64_t u = splitmix64(a.seed, (uint64_t)b * (uint64_t)a.n_shots + (uint64_t)shot);
    uint64_t r = __umul64hi(u, W);
    int64_t base = 0;  // index of the chosen entry at the current level
    for (int k = top; k >= 0; k--) {
        const uint64_t v = k == top ? tv : level_value(k, base * 64 + lane);
        uint64_t incl = v;
        for (int d = 1; d < 64; d <<= 1) {
            uint64_t o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        const uint64_t hit = __ballot(incl > r);
        // the children of the chosen entry sum to its value (> r), so some lane
        // hits; the clamp only keeps indexing in range
        const int sel = hit ? __ffsll((unsigned long long)hit) - 1 : 63;
        const uint64_t before = __shfl(incl - v, sel, 64);
        r -= before;
        base = base * 64 + sel;
    }
    if (lane == 0) *out = (uint64_t)base;
}

// ---------------------------------------------- static sampler workspace
// The level workspace of the sampler for callers that cannot allocate device
// memory (tq_sample_from_state_noalloc): a file-scope device array, one copy
// per GPU, held until the process ends.  In host code its name is only a
// stand-in: kernels get the device address that hipGetSymbolAddress returns
// for the current device, looked up once per device.
static __device__ __align__(256) uint64_t scratch[kStaticLevelEntries];

hipError_t static_levels(uint64_t **ptr)
{
    static std::mutex mu;
    static std::map<int, uint64_t *> addr;  // device -> address of its copy
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> l(mu);
    auto it = addr.find(dev);
    if (it == addr.end()) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        it = addr.emplace(dev, static_cast<uint64_t *>(p)).first;
    }
    *ptr = it->second;
    return hipSuccess;
}

// ------------------------------------------------------- gather, padding
__global__ void k_gather(GatherArgs a)
{
    const int row = blockIdx.y;
    const int b = a.brows ? a.brows[row] : row;
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= a.M) return;
    const uint64_t x = a.bits[(int64_t)b * a.M + m];
    float2 v = make_float2(0.f, 0.f);
    if ((x >> a.n) == 0) v = a.state[(int64_t)(a.rows ? a.rows[row] : row) * a.row_stride + (int64_t)x];
    a.out[(int64_t)b * a.M + m] = v;
}

// out[g, k] = the mean of in[g R + r, k] over r < R (trajectory rows of one
// circuit), summed in fp64 in row order
__global__ void k_row_mean(const float *in, int64_t groups, int32_t R, int32_t K, float *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= groups * K) return;
    const int64_t g = i / K, k = i - g * K;
    const float *p = in + g * R * K + k;
    double s = 0.0;
    for (int32_t r = 0; r < R; r++) s += (double)p[(int64_t)r * K];
    out[i] = (float)(s / R);
}

// ------------------------------------------- batched shift rules
__global__ void k_row_gather(RowGatherArgs a)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= a.count) return;
    const int64_t src = (a.x_begin + r) / a.x_period;
    for (int j = 0; j < a.narrays; j++) a.out[j][r] = a.in[j][src];
}

// Shot counts of the sampled expectation: one wavefront per (launch row,
// term slot), lanes over the shots.  Shot s of term t of observable k in
// counter row e is +1 when (u >> 11) 2^-53 < (1 + e_t) / 2 (fp64, e_t the
// float term expectation clamped to [-1, 1]), u the output number
// ((e K + k) 2^40 + t 2^24 + s) of SplitMix64 from the seed (Sec. "Sampling
// and Expectation Values": a term's shot is the parity of its qubits
// measured in its eigenbasis, +1 with that probability).
__global__ __launch_bounds__(64) void k_sampled_counts(SampledArgs a)
{
    const int64_t w = (int64_t)blockIdx.x + a.w_begin;
    const int r = (int)(w / a.Kt), j = (int)(w - (int64_t)r * a.Kt), lane = threadIdx.x;
    int64_t b = r, e = r;
    if (a.x_period > 0) {
        const int64_t L = a.x_begin + r, src = L / a.x_period;
        b = a.rows[src];
        e = a.ebase[src] + (L - src * a.x_period);
    }
    const int t = a.slot_t[b * a.slot_stride + j];
    if (t < 0) {
        if (lane == 0) a.counts[(int64_t)r * a.Kt + j] = 0;
        return;
    }
    const int k = a.slot_k[b * a.slot_stride + j];
    double ev = (double)a.tv[(int64_t)r * a.Kt + j];
    ev = ev > 1.0 ? 1.0 : ev < -1.0 ? -1.0 : ev;
    const double q = 0.5 * (1.0 + ev);
    const uint64_t base = ((uint64_t)(e * a.K + k) << 40) | ((uint64_t)t << 24);
    uint32_t n = 0;
    for (int sh = lane; sh < a.reps; sh += 64) {
        const uint64_t u = splitmix64(a.seed, base | (uint64_t)sh);
        n += (double)(u >> 11) * 0x1.0p-53 < q;
    }
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
    if (lane == 0) a.counts[(int64_t)r * a.Kt + j] = n;
}

// est = sum over the observable's terms in order of c (identity terms) or
// c (2 n / reps - 1), in fp64 without contractions (the rounding of a plain
// evaluation of that sum), stored as float.
__global__ void k_sampled_combine(SampledArgs a)
{
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)a.nrows * a.K) return;
    const int64_t r = i / a.K;
    const int k = (int)(i - r * a.K);
    int64_t b = r;
    if (a.x_period > 0) b = a.rows[(a.x_begin + r) / a.x_period];
    const int32_t *ob = a.obs_begin + b * a.obs_stride;
    const int32_t *ts = a.term_slot + b * a.term_stride;
    const double *tc = a.term_coeff + b * a.term_stride;
    const double reps = (double)a.reps;
    double est = 0.0;
    for (int t = ob[k]; t < ob[k + 1]; t++) {
        const int j = ts[t];
        if (j < 0) {
            est += tc[t];
            continue;
        }
        const double n = (double)a.counts[r * a.Kt + j];
        est += tc[t] * (2.0 * n / reps - 1.0);
    }
    a.out[i] = (float)est;
}

// Gradients of the batched shift rules (one thread per (group row, symbol)).
__global__ void k_shift_grad(ShiftGradArgs a)
{
    const int srow = blockIdx.x;
    const int s = blockIdx.y * blockDim.x + threadIdx.x;
    if (s >= a.S) return;
    const int64_t b = a.rows[srow];
    const double *scale = a.slot_scale + (a.uniform ? 0 : (int64_t)srow * a.n_slots);
    const float *g = a.upstream + b * a.K;
    double sum = 0.0;
    for (int pi = a.sym_begin[s]; pi < a.sym_begin[s + 1]; pi++) {
        const int p = a.sym_pairs[pi];
        const float *fp = a.f + ((int64_t)srow * a.period + 2 * p) * a.K;
        const float *fm = fp + a.K;
        double d = 0.0;
        for (int k = 0; k < a.K; k++) d += (double)g[k] * ((double)fp[k] - (double)fm[k]);
        const int sl = a.pair_slot[p];
        sum += a.pair_coef[p] * (sl >= 0 ? scale[sl] : 1.0) * d;
    }
    sum *= a.coef_mul;
    a.grad[b * a.S + s] = (float)sum;
}

__global__ __launch_bounds__(256) void k_zero_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    const BatchBlock bb = cget(blocks, blockIdx.x);
    TableArg<ZeroArgs> &a = table_arg<ZeroArgs>(table, bb.arg);
    const int nx = (int)((a.to - a.from + kZeroBlock - 1) / kZeroBlock);
    float2 *st = c.state_out + (int64_t)cget(a.rows, bb.block / nx) * a.row_stride;
    const int64_t from = a.from + (int64_t)(bb.block % nx) * kZeroBlock;
    const int64_t to = from + kZeroBlock < a.to ? from + kZeroBlock : a.to;
    for (int64_t i = from + threadIdx.x; i < to; i += 256) st[i] = make_float2(0.f, 0.f);
}

__global__ void k_zero_tail(float2 *state, int64_t row_stride, const int32_t *rows, int64_t from, int64_t to)
{
    const int row = blockIdx.y;
    const int64_t i = from + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < to) state[(int64_t)rows[row] * row_stride + i] = make_float2(0.f, 0.f);
}

// ------------------------------------------------------- launch wrappers
// Opt-in profiler: launches of the selected kernel are bracketed by a pair
// of HIP events recorded on the launch stream.
namespace prof {
std::mutex mu;
std::string target;
std::vector<std::pair<hipEvent_t, hipEvent_t>> events;

using Scope = ProfScope;
} // namespace prof

ProfScope::ProfScope(const char *name, hipStream_t st) : s(st)
{
    std::lock_guard<std::mutex> l(prof::mu);
    if (prof::target.empty() || prof::target != name) return;
    if (hipEventCreate(&b) != hipSuccess || hipEventCreate(&e) != hipSuccess) {
        b = e = nullptr;
        return;
    }
    (void)hipEventRecord(b, s);
}

ProfScope::~ProfScope()
{
    if (!b) return;
    (void)hipEventRecord(e, s);
    std::lock_guard<std::mutex> l(prof::mu);
    prof::events.emplace_back(b, e);
}

void profile_start(const char *kernel)
{
    std::lock_guard<std::mutex> l(prof::mu);
    prof::target = kernel ? kernel : "";
}

hipError_t profile_read(int64_t *launches, double *total_ms)
{
    std::lock_guard<std::mutex> l(prof::mu);
    double tot = 0;
    hipError_t err = hipSuccess;
    for (auto &pe : prof::events) {
        float ms = 0;
        hipError_t e = hipEventSynchronize(pe.second);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, pe.first, pe.second);
        if (e != hipSuccess) err = e;
        tot += ms;
    }
    *launches = (int64_t)prof::events.size();
    *total_ms = tot;
    for (auto &pe : prof::events) {
        (void)hipEventDestroy(pe.first);
        (void)hipEventDestroy(pe.second);
    }
    prof::events.clear();
    return err;
}

namespace {
template <class K> hipError_t set_lds(K kernel, size_t bytes)
{
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}
} // namespace

hipError_t launch_build_stage(const StageBuildArgs &a, int nrows, hipStream_t s)
{
    if (a.nlist <= 0 || nrows <= 0) return hipSuccess;
    prof::Scope ps("build", s);
    hipLaunchKernelGGL(k_build_stage, dim3(a.nlist, nrows), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_build_derived(const BuildArgs &a, int nrows, int max_list, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    prof::Scope ps("build", s);
    const unsigned blocks = (unsigned)((nrows + 3) / 4);
    if (a.x_copy > 0) hipLaunchKernelGGL(k_copy_source, dim3(blocks), dim3(256), 0, s, a, nrows);
    if (max_list > 0 || a.phase_out >= 0)
        hipLaunchKernelGGL(k_build_list, dim3((unsigned)((nrows + 255) / 256)), dim3(256), 0, s, a, nrows);
    return hipGetLastError();
}

hipError_t launch_build(const BuildArgs &a, int nrows, hipStream_t s)
{
    int n = a.task_end - a.task_begin;
    if (n <= 0 || nrows <= 0) return hipSuccess;
    dim3 grid((n + 255) / 256, nrows);
    prof::Scope ps("build", s);
    hipLaunchKernelGGL(k_build_mats, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

size_t pass_lds_bytes(const TileGeom &g, bool product_init, int nmat)
{
    size_t b = sizeof(float2) * ((size_t)1 << g.t) + sizeof(uint64_t) * ((size_t)1 << g.h) + sizeof(double2) * nmat;
    if (product_init) b += sizeof(double2) * (((size_t)1 << (g.t / 2)) + ((size_t)1 << (g.t - g.t / 2)));
    return b;
}

hipError_t launch_pass(const PassArgs &a, int nrows, hipStream_t s)
{
    size_t lds = pass_lds_bytes(a.g, a.product_init != 0, a.mat_end - a.mat_begin);
    hipError_t e = set_lds(k_pass, lds);
    if (e != hipSuccess) return e;
    prof::Scope ps("pass", s);
    hipLaunchKernelGGL(k_pass, dim3(nrows * a.wg_per_row), dim3(kThreads), lds, s, a);
    return hipGetLastError();
}

size_t pauli_lds_bytes(const TileGeom &g, int k_count, bool partner)
{
    return sizeof(float2) * ((size_t)1 << g.t) * (partner ? 2 : 1) + sizeof(uint64_t) * ((size_t)1 << g.h) +
           sizeof(double) * (4 * kPauliChunk + (size_t)k_count);
}

template <int P>
hipError_t launch_pauli_p(const PauliArgs &a, int nrows, size_t lds, hipStream_t s)
{
    const dim3 grid(nrows * a.wg_per_row);
    if (a.phi) {
        hipError_t e = set_lds(k_pauli<P, true>, lds);
        if (e != hipSuccess) return e;
        prof::Scope ps("pauli", s);
        hipLaunchKernelGGL((k_pauli<P, true>), grid, dim3(kThreads), lds, s, a);
    } else {
        hipError_t e = set_lds(k_pauli<P, false>, lds);
        if (e != hipSuccess) return e;
        prof::Scope ps("pauli", s);
        hipLaunchKernelGGL((k_pauli<P, false>), grid, dim3(kThreads), lds, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_pauli(const PauliArgs &a, int nrows, bool partner, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    const size_t lds = pauli_lds_bytes(a.g, a.k_count, partner);
    switch (a.g.t <= 8 ? 1 : 1 << (a.g.t - 8)) {
    case 1: return launch_pauli_p<1>(a, nrows, lds, s);
    case 2: return launch_pauli_p<2>(a, nrows, lds, s);
    case 4: return launch_pauli_p<4>(a, nrows, lds, s);
    case 8: return launch_pauli_p<8>(a, nrows, lds, s);
    case 16: return launch_pauli_p<16>(a, nrows, lds, s);
    default: return hipErrorInvalidValue;
    }
}

template <int A> hipError_t launch_pauli_diag_a(const DiagArgs &a, int nrows, hipStream_t s)
{
    const size_t lds = sizeof(double) * (size_t)a.k_count;
    hipError_t e = set_lds(k_pauli_diag<A>, lds);
    if (e != hipSuccess) return e;
    prof::Scope ps("pauli", s);
    hipLaunchKernelGGL(k_pauli_diag<A>, dim3(nrows * a.wg_per_row), dim3(kThreads), lds, s, a);
    return hipGetLastError();
}

template <int A> int pauli_diag_slots_a(size_t lds)
{
    // per (device, dynamic LDS size): the query is not free and the answer fixed
    static std::mutex mu;
    static std::map<std::pair<int, size_t>, int> known;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> l(mu);
    auto it = known.find({dev, lds});
    if (it != known.end()) return it->second;
    int per_cu = 0, cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pauli_diag<A>, kThreads, lds) != hipSuccess) return 0;
    return known[{dev, lds}] = per_cu * cus;
}

int pauli_diag_slots(int amax, int k_count)
{
    const size_t lds = sizeof(double) * (size_t)k_count;
    if (amax <= 8) return pauli_diag_slots_a<8>(lds);
    if (amax <= 16) return pauli_diag_slots_a<16>(lds);
    return pauli_diag_slots_a<kDiagClassMax>(lds);
}

hipError_t launch_pauli_diag(const DiagArgs &a, int nrows, int amax, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    if (amax <= 8) return launch_pauli_diag_a<8>(a, nrows, s);
    if (amax <= 16) return launch_pauli_diag_a<16>(a, nrows, s);
    return launch_pauli_diag_a<kDiagClassMax>(a, nrows, s);
}

hipError_t launch_pauli_reduce(const PauliReduceArgs &a, int nrows, hipStream_t s)
{
    if (nrows <= 0 || a.k_count <= 0) return hipSuccess;
    prof::Scope ps("pauli_reduce", s);
    hipLaunchKernelGGL(k_pauli_reduce, dim3(nrows, a.k_count), dim3(256), 0, s, a);
    return hipGetLastError();
}

size_t rev_pass_lds_bytes(const RevArgs &a)
{
    return 2 * sizeof(float2) * ((size_t)1 << a.g.t) + sizeof(uint64_t) * ((size_t)1 << a.g.h) +
           sizeof(double2) * (size_t)(a.mat_end - a.mat_begin) + sizeof(double) * 4 * (size_t)(a.gcount > 0 ? a.gcount : 1);
}

hipError_t launch_rev_pass(const RevArgs &a, int nrows, hipStream_t s)
{
    const size_t lds = rev_pass_lds_bytes(a);
    hipError_t e = set_lds(k_rev_pass, lds);
    if (e != hipSuccess) return e;
    prof::Scope ps("rev_pass", s);
    hipLaunchKernelGGL(k_rev_pass, dim3(nrows * a.wg_per_row), dim3(kThreads), lds, s, a);
    return hipGetLastError();
}

size_t resident_lds_bytes(int n, int nacc, bool adjoint, int waves)
{
    return sizeof(double) * waves * (size_t)nacc + sizeof(float2) * ((size_t)1 << n) * (adjoint ? 2 : 1);
}

hipError_t launch_resident(const ResArgs &a, int nrows, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    size_t lds = resident_lds_bytes(a.n, a.nacc, a.grad != nullptr);
    hipError_t e = set_lds(k_resident, lds);
    if (e != hipSuccess) return e;
    prof::Scope ps("resident", s);
    hipLaunchKernelGGL(k_resident, dim3(nrows), dim3(kThreads), lds, s, a);
    return hipGetLastError();
}

template <class K>
hipError_t launch_batch_k(K kernel, const char *name, int threads, const void *table, const BatchBlock *blocks,
                          int nblocks, size_t lds, const ResCall &c, hipStream_t s)
{
    hipError_t e = set_lds(kernel, lds);
    if (e != hipSuccess) return e;
    prof::Scope ps(name, s);
    hipLaunchKernelGGL(kernel, dim3((unsigned)nblocks), dim3(threads), lds, s, table, blocks, c);
    return hipGetLastError();
}

template <int P>
hipError_t launch_pauli_batch(bool phi, const void *table, const BatchBlock *blocks, int nblocks, size_t lds,
                              const ResCall &c, hipStream_t s)
{
    return phi ? launch_batch_k(k_pauli_batch<P, true>, "pauli", 256, table, blocks, nblocks, lds, c, s)
               : launch_batch_k(k_pauli_batch<P, false>, "pauli", 256, table, blocks, nblocks, lds, c, s);
}

hipError_t launch_batch(int kind, const void *table, const BatchBlock *blocks, int nblocks, size_t lds, int threads,
                        int p, bool phi, const ResCall &c, hipStream_t s)
{
    if (nblocks <= 0) return hipSuccess;
    switch (kind) {
    case BK_BUILD: return launch_batch_k(k_build_batch, "build", 256, table, blocks, nblocks, lds, c, s);
    case BK_STAGE: return launch_batch_k(k_stage_batch, "build", 64, table, blocks, nblocks, lds, c, s);
    case BK_RESIDENT:
        if (threads == 1024)
            return launch_batch_k(k_resident_batch<1024>, "resident", 1024, table, blocks, nblocks, lds, c, s);
        return launch_batch_k(k_resident_batch<256>, "resident", 256, table, blocks, nblocks, lds, c, s);
    case BK_PASS: return launch_batch_k(k_pass_batch, "pass", 256, table, blocks, nblocks, lds, c, s);
    case BK_PAULI:
        switch (p) {
        case 1: return launch_pauli_batch<1>(phi, table, blocks, nblocks, lds, c, s);
        case 2: return launch_pauli_batch<2>(phi, table, blocks, nblocks, lds, c, s);
        case 4: return launch_pauli_batch<4>(phi, table, blocks, nblocks, lds, c, s);
        case 8: return launch_pauli_batch<8>(phi, table, blocks, nblocks, lds, c, s);
        case 16: return launch_pauli_batch<16>(phi, table, blocks, nblocks, lds, c, s);
        default: return hipErrorInvalidValue;
        }
    case BK_PAULI_REDUCE:
        return launch_batch_k(k_pauli_reduce_batch, "pauli_reduce", 256, table, blocks, nblocks, lds, c, s);
    case BK_REV: return launch_batch_k(k_rev_batch, "rev_pass", 256, table, blocks, nblocks, lds, c, s);
    case BK_GRAD_REDUCE: return launch_batch_k(k_grad_reduce_batch, "grad_reduce", 256, table, blocks, nblocks, lds, c, s);
    case BK_ZERO: return launch_batch_k(k_zero_batch, "zero", 256, table, blocks, nblocks, lds, c, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_grad_reduce(const GradReduceArgs &a, int nrows, hipStream_t s)
{
    prof::Scope ps("grad_reduce", s);
    hipLaunchKernelGGL(k_grad_reduce, dim3(nrows), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_sample(const SampArgs &a, int nrows, hipStream_t s)
{
    if (nrows <= 0) return hipSuccess;
    if (a.nlev >= 1) {
        {
            prof::Scope ps("samp_l1", s);
            // eight lanes per group of 64 amplitudes, at most 8192 workgroups
            // over all rows (grid-stride beyond)
            const int64_t blocks = std::min<int64_t>((a.count[1] * 8 + 255) / 256, std::max(1, 8192 / nrows));
            hipLaunchKernelGGL(k_samp_l1, dim3((unsigned)blocks, nrows), dim3(256), 0, s, a);
        }
        for (int k = 1; k < a.nlev; k++)
            hipLaunchKernelGGL(k_samp_up, dim3((unsigned)((a.count[k + 1] + 3) / 4), nrows), dim3(256), 0, s, a, k);
    }
    if (a.n_shots > 0) {
        prof::Scope ps("samp_shots", s);
        hipLaunchKernelGGL(k_samp_shots, dim3((unsigned)((a.n_shots + 3) / 4), nrows), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_gather(const GatherArgs &a, int nrows, hipStream_t s)
{
    if (a.M <= 0 || nrows <= 0) return hipSuccess;
    prof::Scope ps("gather", s);
    hipLaunchKernelGGL(k_gather, dim3((unsigned)((a.M + 255) / 256), nrows), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_row_mean(const float *in, int64_t groups, int32_t R, int32_t K, float *out, hipStream_t s)
{
    const int64_t n = groups * K;
    if (n <= 0) return hipSuccess;
    prof::Scope ps("row_mean", s);
    hipLaunchKernelGGL(k_row_mean, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, in, groups, R, K, out);
    return hipGetLastError();
}

hipError_t launch_row_gather(const RowGatherArgs &a, hipStream_t s)
{
    if (a.count <= 0 || a.narrays <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_row_gather, dim3((unsigned)((a.count + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_sampled(const SampledArgs &a, hipStream_t s)
{
    if (a.nrows <= 0 || a.K <= 0) return hipSuccess;
    if (a.Kt > 0) {
        prof::Scope ps("sampled_counts", s);
        // one wavefront per (row, term slot), at most 2^30 per launch
        const int64_t waves = (int64_t)a.nrows * a.Kt;
        for (int64_t w0 = 0; w0 < waves; w0 += (int64_t)1 << 30) {
            SampledArgs c = a;
            c.w_begin = w0;
            hipLaunchKernelGGL(k_sampled_counts, dim3((unsigned)std::min<int64_t>(waves - w0, (int64_t)1 << 30)),
                               dim3(64), 0, s, c);
        }
    }
    const int64_t n = (int64_t)a.nrows * a.K;
    hipLaunchKernelGGL(k_sampled_combine, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_shift_grad(const ShiftGradArgs &a, int nrows, hipStream_t s)
{
    if (nrows <= 0 || a.S <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_shift_grad, dim3((unsigned)nrows, (unsigned)((a.S + 63) / 64)), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_zero_tail(float2 *state, int64_t row_stride, const int32_t *rows, int nrows, int64_t from, int64_t to,
                            hipStream_t s)
{
    if (to <= from || nrows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_tail, dim3((unsigned)((to - from + 255) / 256), nrows), dim3(256), 0, s, state,
                       row_stride, rows, from, to);
    return hipGetLastError();
}

} // namespace tq
