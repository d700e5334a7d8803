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
__host__ __device__ __forceinline__ constexpr cd C(double x, double y) { return cd{x, y}; }
__host__ __device__ __forceinline__ cd cdmul(cd a, cd b) { return cd{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__host__ __device__ __forceinline__ cd cdadd(cd a, cd b) { return cd{a.x + b.x, a.y + b.y}; }

// sin and cos of x, or of pi x (half_turns).  Every lane of a builder
// wavefront needs one and a lone wavefront runs at the speed of its
// instruction stream, so both kinds share one short straight-line path: the
// argument is reduced to y + yl, |y| <= pi/4, by k quarter turns (exactly for
// pi x; for x by pi/2 in two parts, with k P1 exact under FMA while |x| <
// 2^20; larger arguments take the library's reduction), then the Taylor series
// (remainders y^19/19! < 1e-19 and y^18/18! < 3e-18).
__host__ __device__ __forceinline__ void sincos_of(double x, bool half_turns, double *s, double *c)
{
    const double k = half_turns ? std::rint(2.0 * x) : std::rint(x * 0.63661977236758134308);
    double y, yl;
    if (half_turns) {
        const double r = std::fma(-0.5, k, x);
        y = r * 3.14159265358979311600;
        yl = std::fma(r, 3.14159265358979311600, -y) + r * 1.22464679914735320717e-16;
    } else {
        const double r = std::fma(-k, 1.57079632679489655800, x);
        y = std::fma(-k, 6.12323399573676603587e-17, r);
        yl = std::fma(-k, 6.12323399573676603587e-17, r - y);
    }
    const double z = y * y;
    double ps = 1.0 / 355687428096000.0, pc = 1.0 / 20922789888000.0;  // 1/17!, 1/16!
    ps = std::fma(ps, z, -1.0 / 1307674368000.0);
    pc = std::fma(pc, z, -1.0 / 87178291200.0);
    ps = std::fma(ps, z, 1.0 / 6227020800.0);
    pc = std::fma(pc, z, 1.0 / 479001600.0);
    ps = std::fma(ps, z, -1.0 / 39916800.0);
    pc = std::fma(pc, z, -1.0 / 3628800.0);
    ps = std::fma(ps, z, 1.0 / 362880.0);
    pc = std::fma(pc, z, 1.0 / 40320.0);
    ps = std::fma(ps, z, -1.0 / 5040.0);
    pc = std::fma(pc, z, -1.0 / 720.0);
    ps = std::fma(ps, z, 1.0 / 120.0);
    pc = std::fma(pc, z, 1.0 / 24.0);
    ps = std::fma(ps, z, -1.0 / 6.0);
    const double w = 0.5 * z, c0 = 1.0 - w;
    const double sy = y + std::fma(y * z, ps, std::fma(-w, yl, yl));
    const double cy = c0 + (((1.0 - c0) - w) + std::fma(z * z, pc, -y * yl));
    // k mod 4 without an integer conversion that could overflow
    const double q4 = k - 4.0 * std::floor(0.25 * k);
    const bool odd = q4 == 1.0 || q4 == 3.0;
    const double ss = odd ? cy : sy, cc = odd ? sy : cy;
    *s = q4 >= 2.0 ? -ss : ss;
    *c = q4 == 1.0 || q4 == 2.0 ? -cc : cc;
    // (infinities and NaN take this path as well)
    if (!half_turns && !(std::fabs(x) < 1048576.0)) {
#if defined(__HIP_DEVICE_COMPILE__)
        sincos(x, s, c);
#else
        *s = std::sin(x);
        *c = std::cos(x);
#endif
    }
}

// The angle a gate's matrix is written in: eta / 2 (RX, RY), eta (RZ, RZZ,
// fSim's theta), pi t / 2 (X^t, Y^t, XX^t, YY^t) or pi t (Z^t, CZ^t, CNOT^t,
// ZZ^t); pi / 4 for the gates without one, whose tables use cos and sin of it
// as 1/sqrt(2).  deriv: times the derivative of the angle by eta, which every
// entry of a derivative carries.
constexpr uint32_t op_set() { return 0; }
template <class... T> constexpr uint32_t op_set(int op, T... rest) { return (1u << op) | op_set(rest...); }
constexpr uint32_t kRadian = op_set(OP_RX, OP_RY, OP_RZ, OP_RZZ, OP_FSIM);
constexpr uint32_t kTurns = op_set(OP_XPOW, OP_YPOW, OP_XXPOW, OP_YYPOW, OP_ZPOW, OP_CZPOW, OP_CNOTPOW, OP_ZZPOW);
constexpr uint32_t kHalfAngle = op_set(OP_RX, OP_RY, OP_XPOW, OP_YPOW, OP_XXPOW, OP_YYPOW);
__host__ __device__ __forceinline__ void gate_angle(int op, double eta, bool deriv, double *s, double *c)
{
    const uint32_t bit = op < 32 ? 1u << op : 0u;
    const bool turns = (bit & kTurns) != 0, plain = (bit & (kRadian | kTurns)) == 0;
    const double h = bit & kHalfAngle ? 0.5 : 1.0;
    sincos_of(h * eta, turns, s, c);
    if (plain) *s = *c = 0.70710678118654752440;
    if (deriv) {
        const double dh = turns ? h * 3.14159265358979323846 : h;
        *s *= dh;
        *c *= dh;
    }
}

// The tables: matrices and derivatives, entries linear in 1, c and s with
// coefficients in halves (see GateCodes).  m: row-major, zero-initialised;
// the dimension is returned, 0 if the gate has none in that form.
// MATRIX1/MATRIX2 and fSim's second parameter (entry 15) are not in them.
constexpr int gate_matrix(int op, int form, double s, double c, cd *m)
{
    switch (op) {
    case OP_H: m[0] = C(c, 0); m[1] = C(c, 0); m[2] = C(c, 0); m[3] = C(-c, 0); return 2;
    case OP_X: m[1] = C(1, 0); m[2] = C(1, 0); return 2;
    case OP_Y: m[1] = C(0, -1); m[2] = C(0, 1); return 2;
    case OP_Z: m[0] = C(1, 0); m[3] = C(-1, 0); return 2;
    case OP_RX: case OP_XPOW: case OP_SQRTX:
        m[0] = C(c, 0); m[1] = C(0, -s); m[2] = C(0, -s); m[3] = C(c, 0); return 2;
    case OP_RY: case OP_YPOW: case OP_SQRTY:
        m[0] = C(c, 0); m[1] = C(-s, 0); m[2] = C(s, 0); m[3] = C(c, 0); return 2;
    case OP_RZ: case OP_ZPOW: m[0] = C(1, 0); m[3] = C(c, s); return 2;
    case OP_SQRTW:
        // W^{1/2} = e^{i pi/4} (cos(pi/4) I - i sin(pi/4) W) with W = [[0, e^{-i pi/4}],
        // [e^{i pi/4}, 0]]: without the phase, r I - i r W with r = 1/sqrt(2)
        // (real diagonal; -i r e^{-/+ i pi/4} = (-1 -/+ i)/2 off it)
        m[0] = m[3] = C(c, 0); m[1] = C(-0.5, -0.5); m[2] = C(0.5, -0.5);
        return 2;
    case OP_CZ: m[0] = m[5] = m[10] = C(1, 0); m[15] = C(-1, 0); return 4;
    case OP_CZPOW: m[0] = m[5] = m[10] = C(1, 0); m[15] = C(c, s); return 4;
    case OP_CNOT:
        if (form == FORM_CBLOCK) { m[1] = m[2] = C(1, 0); return 2; }
        m[0] = m[5] = C(1, 0); m[11] = m[14] = C(1, 0); return 4;
    case OP_CNOTPOW: {
        const cd p = C(0.5 * (1 + c), 0.5 * s), q = C(0.5 * (1 - c), -0.5 * s);
        if (form == FORM_CBLOCK) { m[0] = m[3] = p; m[1] = m[2] = q; return 2; }
        m[0] = m[5] = C(1, 0); m[10] = m[15] = p; m[11] = m[14] = q; return 4;
    }
    case OP_XXPOW:  // cos I - i sin XX; XX couples 00 with 11 and 01 with 10, all with +1
        m[0] = m[5] = m[10] = m[15] = C(c, 0);
        m[3] = m[6] = m[9] = m[12] = C(0, -s);
        return 4;
    case OP_YYPOW:  // cos I - i sin YY; YY = -|11><00| - |00><11| + |10><01| + |01><10|
        m[0] = m[5] = m[10] = m[15] = C(c, 0);
        m[3] = m[12] = C(0, s);
        m[6] = m[9] = C(0, -s);
        return 4;
    case OP_ZZPOW: case OP_RZZ: m[0] = m[15] = C(1, 0); m[5] = m[10] = C(c, s); return 4;
    case OP_FSIM: m[0] = C(1, 0); m[5] = m[10] = C(c, 0); m[6] = m[9] = C(0, -s); return 4;
    case OP_SWAP: m[0] = m[6] = m[9] = m[15] = C(1, 0); return 4;
    }
    return 0;
}
// derivatives of the matrices (as built, without their left-out phase) with
// respect to parameter `which`; s and c carry the derivative of the angle
constexpr int gate_deriv(int op, int form, int which, double s, double c, cd *m)
{
    switch (op) {
    case OP_RX: case OP_XPOW: m[0] = C(-s, 0); m[1] = C(0, -c); m[2] = C(0, -c); m[3] = C(-s, 0); return 2;
    case OP_RY: case OP_YPOW: m[0] = C(-s, 0); m[1] = C(-c, 0); m[2] = C(c, 0); m[3] = C(-s, 0); return 2;
    case OP_RZ: case OP_ZPOW: m[3] = C(-s, c); return 2;
    case OP_CZPOW: m[15] = C(-s, c); return 4;
    case OP_CNOTPOW: {
        const cd p = C(-0.5 * s, 0.5 * c), q = C(0.5 * s, -0.5 * c);
        if (form == FORM_CBLOCK) { m[0] = m[3] = p; m[1] = m[2] = q; return 2; }
        m[10] = m[15] = p; m[11] = m[14] = q; return 4;
    }
    case OP_XXPOW: m[0] = m[5] = m[10] = m[15] = C(-s, 0); m[3] = m[6] = m[9] = m[12] = C(0, -c); return 4;
    case OP_YYPOW:  // YY: -1 on (00, 11) and (11, 00), +1 on (01, 10) and (10, 01)
        m[0] = m[5] = m[10] = m[15] = C(-s, 0); m[3] = m[12] = C(0, c); m[6] = m[9] = C(0, -c); return 4;
    case OP_ZZPOW: case OP_RZZ: m[5] = m[10] = C(-s, c); return 4;
    case OP_FSIM:
        if (which == 0) { m[5] = m[10] = C(-s, 0); m[6] = m[9] = C(0, -c); }
        return 4;
    }
    return 0;
}
// fSim's entry 15: e^{-i phi}, or its derivative -i e^{-i phi}, from sin and cos of phi
__host__ __device__ __forceinline__ cd fsim_corner(double s, double c, bool deriv, int which)
{
    return !deriv ? C(c, -s) : which == 1 ? C(-s, -c) : C(0, 0);
}

// The tables as the builder reads them: an entry's six coefficients (real,
// then imaginary part; of 1, c and s) in halves, four signed bits each.  The
// lanes of a wavefront build different gates' matrices: a switch runs its
// cases one after another, each with instruction fetches that miss (measured
// on a lone wavefront: 2600 instructions, 60% of the time waiting), a table
// makes every entry the same few instructions.  Row: (derivative by the first,
// second parameter or none; form; qubits swapped; op).
struct GateCodes {
    uint32_t e[3][2][2][32][16];
};
constexpr uint32_t half_units(double a, double b, double c)
{
    const double v[3] = {2 * a, 2 * b, 2 * c};
    uint32_t r = 0;
    for (int i = 0; i < 3; i++) r |= ((uint32_t)(int)v[i] & 15u) << (4 * i);
    return r;
}
constexpr GateCodes gate_codes()
{
    GateCodes t{};
    for (int d = 0; d < 3; d++)
        for (int form = 0; form < 2; form++)
            for (int sw = 0; sw < 2; sw++)
                for (int op = 0; op < 32; op++) {
                    cd m[3][16] = {};
                    int dim = 0;
                    for (int b = 0; b < 3; b++) {
                        const double s = b == 2 ? 1 : 0, c = b == 1 ? 1 : 0;
                        dim = d ? gate_deriv(op, form, d - 1, s, c, m[b]) : gate_matrix(op, form, s, c, m[b]);
                    }
                    for (int i = 0; i < dim; i++)
                        for (int j = 0; j < dim; j++) {
                            // (reversed qubit order: |ab> -> |ba>)
                            const int pi = sw && dim == 4 && (i == 1 || i == 2) ? 3 - i : i;
                            const int pj = sw && dim == 4 && (j == 1 || j == 2) ? 3 - j : j;
                            const int k = i * dim + j;
                            t.e[d][form][sw][op][pi * dim + pj] =
                                half_units(m[0][k].x, m[1][k].x - m[0][k].x, m[2][k].x - m[0][k].x) |
                                half_units(m[0][k].y, m[1][k].y - m[0][k].y, m[2][k].y - m[0][k].y) << 12;
                        }
                }
    return t;
}
__device__ const GateCodes kGateCodes = gate_codes();

// The matrix of a row of codes at c and s.  A coefficient 0 leaves a
// non-finite angle out of its entry.
__device__ __forceinline__ double code_part(uint32_t q, double c2, double s2)
{
    const double k0 = (double)((int32_t)(q << 28) >> 28), kc = (double)((int32_t)(q << 24) >> 28),
                 ks = (double)((int32_t)(q << 20) >> 28);
    return fma(kc, c2, fma(ks, s2, 0.5 * k0));
}
template <int N> __device__ __forceinline__ void code_values(const uint32_t *q, double s, double c, cd *g)
{
    const double c2 = 0.5 * c, s2 = 0.5 * s;
#pragma unroll
    for (int i = 0; i < N; i++) g[i] = C(code_part(q[i], c2, s2), code_part(q[i] >> 12, c2, s2));
    if (!(fabs(s) + fabs(c) < 1e300)) {
#pragma unroll
        for (int i = 0; i < N; i++) {
            if (!(q[i] & 0xff0u)) g[i].x = 0.5 * (double)((int32_t)(q[i] << 28) >> 28);
            if (!((q[i] >> 12) & 0xff0u)) g[i].y = 0.5 * (double)((int32_t)(q[i] << 16) >> 28);
        }
    }
}
// entries at(0 .. 3) of a row into g
template <class At>
__device__ __forceinline__ void code_entries4(const uint32_t *code, At at, double s, double c, cd *g)
{
    uint32_t q[4];
#pragma unroll
    for (int i = 0; i < 4; i++) q[i] = code[at(i)];
    code_values<4>(q, s, c, g);
}
// All sixteen, N at a time: fewer as more of them are held, so that the
// unpacked coefficients stay within the 256 registers of two wavefronts per
// SIMD.  All at once the builder took 310, one wavefront; gradients with dense
// 4x4 products, the builder alone: 16384 rows of 3 qubits 1005 -> 577 us, 16384
// of 8 qubits 694 -> 240, 1024 of 8 qubits 58 -> 42, a row of 13 qubits 17.7 ->
// 18.3.
template <int N, int... Rest>
__device__ __forceinline__ void code_steps(const uint32_t *q, double s, double c, cd *g)
{
    __builtin_amdgcn_sched_barrier(0);
    code_values<N>(q, s, c, g);
    if constexpr (sizeof...(Rest) > 0) code_steps<Rest...>(q + N, s, c, g + N);
    else __builtin_amdgcn_sched_barrier(0);
}

int gate_table_host(int op, const double *eta, const double *ex, int form, int deriv, int which, double *out)
{
    cd m[16];
    for (int i = 0; i < 16; i++) m[i] = C(0, 0);
    double s, c;
    gate_angle(op, eta[0], deriv != 0, &s, &c);
    int d = deriv ? gate_deriv(op, form, which, s, c, m) : gate_matrix(op, form, s, c, m);
    if (op == OP_FSIM) {
        gate_angle(op, eta[1], deriv != 0, &s, &c);
        m[15] = fsim_corner(s, c, deriv != 0, which);
    }
    if (!deriv && (op == OP_MATRIX1 || op == OP_MATRIX2)) {
        d = op == OP_MATRIX1 ? 2 : 4;
        for (int i = 0; i < d * d; i++) m[i] = C(ex[2 * i], ex[2 * i + 1]);
    }
    for (int i = 0; i < d * d; i++) {
        out[2 * i] = m[i].x;
        out[2 * i + 1] = m[i].y;
    }
    return d;
}

// entry i of a 4x4 matrix under reversed qubit order (|ab> -> |ba>)
__device__ __forceinline__ int swapped_entry(int i)
{
    const int sw = 0xd8;  // 0, 2, 1, 3
    return ((sw >> (2 * (i >> 2))) & 3) * 4 + ((sw >> (2 * (i & 3))) & 3);
}

// Where the builder finds one batch row's parameters.
struct BuildCtx {
    const MemberDev *members;
    const GateDev *gates;
    const int32_t *slot_sym;
    const double *scale, *off;  // this row's scale and offset per slot
    const double *explicit_mats;
    const float *theta;         // this row's symbol values
    uint64_t noise_seed;        // channels: the row's trajectory draws
    int64_t b;                  // batch row
    const ShiftDev *shift;      // derived rows: the row's parameter moves (else NULL)
    double eps;                 // symbol moves are dtheta x eps
    bool phased;                // the row's global phase is kept (derived rows: not)
    const uint32_t *frame;      // the row's Pauli frame (NULL: none)
    int frame_words;
    __device__ __forceinline__ bool flipped(int bit) const
    {
        return frame && bit >= 0 && ((frame[bit >> 5] >> (bit & 31)) & 1u);
    }
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
struct SlotLoad {
    double scale, off;
    float theta;
};
__device__ __forceinline__ SlotLoad slot_load(const BuildCtx &c, int slot, int sy)
{
    SlotLoad l{0.0, 0.0, 0.0f};
    if (slot >= 0) {
        l.scale = c.scale[slot];
        l.off = c.off[slot];
        if (sy >= 0) l.theta = c.theta[sy];
    }
    return l;
}
__device__ __forceinline__ double slot_value(const BuildCtx &c, int slot, int sy, const SlotLoad &l)
{
    if (sy < 0) return l.off;
    if (!c.shift) return fma(l.scale, (double)l.theta, l.off);
    const ShiftDev &x = *c.shift;
    const double th = sy == x.sym ? fma(x.dtheta, c.eps, (double)l.theta) : (double)l.theta;
    const double eta = fma(l.scale, th, l.off);
    return slot == x.slot[0] ? eta + x.delta[0] : slot == x.slot[1] ? eta + x.delta[1] : eta;
}
__device__ __forceinline__ double slot_value(const BuildCtx &c, int slot, int sy)
{
    return slot_value(c, slot, sy, slot_load(c, slot, sy));
}

// Half turns of a forward rotation task: its angle phi (the sum over its
// members, all about one axis), the matrix being cos phi I - i sin phi G, in
// units of pi and modulo 2, so that the sum keeps its parity however large the
// parameters are.  half_turns: a member's phi / pi at its parameter eta, in
// [-1, 1].  Where eta / (2 pi) may have lost its fraction it comes from the
// angle's sine s and cosine c, asin to m^5 within 1e-3 (the shears hold for any
// cosine well above -1, so the parity may be off near an odd quarter turn).  One
// lane counts the tasks of other blocks again, so every operation is rounded on
// its own (no product is left to be contracted into a sum): the two counts are
// the same bit for bit.
constexpr double kTurnsExact = 1099511627776.0;  // 2^40
__device__ __forceinline__ bool far_turned(const MemberDev &gd, double eta)
{
    return (gd.op == OP_RX || gd.op == OP_RY) && !(fabs(eta) < kTurnsExact);
}
__device__ __forceinline__ double mod2(double t) { return fma(-2.0, rint(0.5 * t), t); }
__device__ __forceinline__ double half_turns(const MemberDev &gd, double eta, double s, double c)
{
    if (gd.slot[0] < 0) return 0.25;  // sqrt X, sqrt Y: G^(1/2)
    if (far_turned(gd, eta)) {
        const bool steep = fabs(s) > fabs(c);
        const double m = fmin(fabs(s), fabs(c)), z = m * m;
        const double k = fma(z, fma(z, 0.0239, 0.0531), 0.3183);  // (1 + z / 6 + 3 z^2 / 40) / pi
        return copysign(fma(steep == (c < 0.0) ? m : -m, k, steep ? 0.5 : c < 0.0 ? 1.0 : 0.0), s);
    }
    return mod2(gd.op == OP_RX || gd.op == OP_RY ? eta * (0.5 / 3.14159265358979323846) : 0.5 * eta);
}
__device__ __forceinline__ int odd_turns(double phi) { return fabs(mod2(phi)) > 0.5; }
__device__ __forceinline__ int rot_turns(const BuildTask &bt, const BuildCtx &c)
{
    double phi = 0.0;
    for (int mi = 0; mi < bt.mem_count; mi++) {
        const MemberDev gd = c.members[bt.mem_begin + mi];
        double eta = slot_value(c, gd.slot[0], gd.sym[0]);
        if (c.flipped(gd.flip)) eta = -eta;
        double sn = 0.0, cs = 1.0;
        if (far_turned(gd, eta)) gate_angle(gd.op, eta, false, &sn, &cs);
        phi += half_turns(gd, eta, sn, cs);
    }
    return odd_turns(phi);
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

// The matrix product of one member, g, and the members before it (column by
// column: column j of g acc needs column j of acc alone).
template <int D> __device__ __forceinline__ void apply_left(const cd *g, cd *acc)
{
#pragma unroll
    for (int j = 0; j < D; j++) {
        cd t[D];
#pragma unroll
        for (int i = 0; i < D; i++) {
            t[i] = C(0, 0);
#pragma unroll
            for (int k = 0; k < D; k++) t[i] = cdadd(t[i], cdmul(g[i * D + k], acc[k * D + j]));
        }
#pragma unroll
        for (int i = 0; i < D; i++) acc[i * D + j] = t[i];
    }
}
// A Pauli channel's (this row's draw) or a frame's (X^x Z^z of qubit slot0)
// Pauli.
__device__ __forceinline__ void pauli_matrix(const BuildCtx &c, const MemberDev &gd, cd *g)
{
    int x, z;
    bool y = false;
    if (gd.op == OP_FRAME) {
        x = (c.frame[c.frame_words - 3] >> gd.slot[0]) & 1u;
        z = (c.frame[c.frame_words - 2] >> gd.slot[0]) & 1u;
    } else {
        const int k = channel_pick(c.noise_seed, c.b, gd.chan, c.off + gd.slot[0]);
        x = k == 1 || k == 2;
        z = k == 2 || k == 3;
        y = k == 2;  // Y = i X Z
    }
    const double sg = z ? -1.0 : 1.0;
    g[0] = C(x ? 0.0 : 1.0, 0);
    g[1] = C(x && !y ? sg : 0.0, y ? sg : 0.0);
    g[2] = C(x && !y ? 1.0 : 0.0, y ? 1.0 : 0.0);
    g[3] = C(x ? 0.0 : sg, 0);
}

// One build task for one row: symbol resolution eta = scale*theta + offset
// and the fused product / dagger / derivative, all in float64.  A lone
// wavefront is bound by the fetch of the code it runs through, so the shapes
// that nearly all tasks have share one path of four entries: 2x2 matrices, the
// pairs a I + b P (their product is that of the middle blocks [[a, b], [b,
// a]]) and diagonals of 4x4 matrices; other 4x4 matrices go through 16.
// Measured, kernel alone, against a switch over the gates in each lane with
// four dependent loads per member: 987 rows of 7 qubits 12.6 -> 6.6 us; the
// shifted rows of 823 rows of 3 qubits 203 -> 53 us, 11 rows of 6 qubits 8.1 ->
// 7.5 us.
// Returns 1 when its shears leave out a sign that belongs to the row's phase.
template <bool FULL> __device__ __forceinline__ int build_task(const BuildTask &bt, const BuildCtx &c, double2 *out)
{
    constexpr int NA = FULL ? 16 : 4;
    cd acc[NA];
    const bool two = bt.dim == 2, pair = !two && (bt.diag == 2 || bt.diag == 3), diag4 = !two && bt.diag == 1;
    const bool small = !FULL || two || pair || diag4, deriv = bt.kind == BT_DERIV, first_only = bt.kind != BT_PRODUCT;
    const uint32_t at4 = two ? 0x3210u : pair ? 0xa965u : 0xfa50u;
    // (the sign of a phase-keeping row's forward rotation comes from its angle)
    const bool turns = bt.kind == BT_PRODUCT && bt.which != BX_NONE && c.phased;
    double phi = 0.0;
    // (a task without members is the identity: a qubit no gate prepares)
#pragma unroll
    for (int i = 0; i < NA; i++) acc[i] = C((small ? i == 0 || i == 3 : i % 5 == 0) ? 1 : 0, 0);
    const int last = bt.mem_begin + bt.mem_count - 1;
    MemberDev next{};
    next.slot[0] = -1;
    if (bt.mem_count > 0) next = c.members[bt.mem_begin];
    SlotLoad loaded = slot_load(c, next.op == OP_FRAME ? -1 : next.slot[0], next.sym[0]);
    for (int mi = 0; mi < bt.mem_count; mi++) {
        // the next member's loads run under this one's arithmetic
        const MemberDev gd = next;
        next = c.members[min(bt.mem_begin + mi + 1, last)];
        double eta = slot_value(c, gd.slot[0], gd.sym[0], loaded);
        if (c.flipped(gd.flip)) eta = -eta;
        const uint32_t *code = kGateCodes.e[deriv ? 1 + bt.which : 0][gd.form][gd.swapped][gd.op & 31];
        const double *ex = gd.explicit_ >= 0 ? c.explicit_mats + 32 * gd.explicit_ : nullptr;
        double sn = 0.0, cs = 1.0;
        cd corner = C(0, 0);
        for (int j = gd.op == OP_FSIM ? 1 : 0; j >= 0; j--) {
            gate_angle(gd.op, j ? slot_value(c, gd.slot[1], gd.sym[1]) : eta, deriv, &sn, &cs);
            if (j) corner = fsim_corner(sn, cs, deriv, bt.which);
        }
        if (turns) phi += half_turns(gd, eta, sn, cs);
        loaded = slot_load(c, next.op == OP_FRAME ? -1 : next.slot[0], next.sym[0]);
        if (small) {
            cd g[4];
            code_entries4(code, [&](int i) { return (at4 >> (4 * i)) & 15u; }, sn, cs, g);
            if (ex) {
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int k = (at4 >> (4 * i)) & 15u, e = gd.swapped && !two ? swapped_entry(k) : k;
                    g[i] = C(ex[2 * e], ex[2 * e + 1]);
                }
            }
            if (gd.op == OP_FSIM && diag4) g[3] = corner;
            if (gd.op == OP_PCHAN || gd.op == OP_FRAME) pauli_matrix(c, gd, g);
            if (mi == 0 || first_only) {
#pragma unroll
                for (int i = 0; i < 4; i++) acc[i] = g[i];
            } else if (diag4) {
#pragma unroll
                for (int i = 0; i < 4; i++) acc[i] = cdmul(g[i], acc[i]);
            } else {
                apply_left<2>(g, acc);
            }
        } else if constexpr (FULL) {
            cd g[16];
            uint32_t q[16];
#pragma unroll
            for (int i = 0; i < 16; i++) q[i] = code[i];
            code_steps<4, 4, 2, 2, 1, 1, 1, 1>(q, sn, cs, g);
            if (ex) {
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    const int e = gd.swapped ? swapped_entry(i) : i;
                    g[i] = C(ex[2 * e], ex[2 * e + 1]);
                }
            }
            if (gd.op == OP_FSIM) g[15] = corner;
            if (mi == 0 || first_only) {
#pragma unroll
                for (int i = 0; i < 16; i++) acc[i] = g[i];
            } else {
                apply_left<4>(g, acc);
            }
        }
    }
    if (bt.kind == BT_DAGGER) {
#pragma unroll
        for (int i = 0; i < NA; i++) acc[i].y = -acc[i].y;
        if (two || pair) {
            const cd t = acc[1];
            acc[1] = acc[2];
            acc[2] = t;
        } else if constexpr (FULL) {
            if (!small) {
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < i; j++) {
                    const cd t = acc[i * 4 + j];
                    acc[i * 4 + j] = acc[j * 4 + i];
                    acc[j * 4 + i] = t;
                }
            }
        }
    }
    if (small) {
        // a pair stores (a, b), a 2x2 diagonal its entries 0 and 3
        const bool d2 = two && bt.diag != 0;
        out[0] = make_double2(acc[0].x, acc[0].y);
        out[1] = d2 ? make_double2(acc[3].x, acc[3].y) : make_double2(acc[1].x, acc[1].y);
        if (!d2 && !pair) {
            out[2] = make_double2(acc[2].x, acc[2].y);
            out[3] = make_double2(acc[3].x, acc[3].y);
        }
    } else if constexpr (FULL) {
        if (bt.diag == 4) {
            // excitation preserving: |00> phase, the (|01>, |10>) block, |11> phase
            const int ix[6] = {0, 5, 6, 9, 10, 15};
#pragma unroll
            for (int i = 0; i < 6; i++) out[i] = make_double2(acc[ix[i]].x, acc[ix[i]].y);
        } else {
#pragma unroll
            for (int i = 0; i < 16; i++) out[i] = make_double2(acc[i].x, acc[i].y);
        }
    }
    if (deriv || bt.which == BX_NONE) return 0;
    const double cr = acc[0].x, sr = bt.which == BX_REAL ? acc[2].x : -acc[2].y;
    const bool odd = turns ? odd_turns(phi) != 0 : cr < 0.0;
    out[two ? 4 : 2] = shear_of(cr, sr, odd);
    return turns && odd;
}

// --------------------------------------------------------- Pauli frames
// The frame of batch row b into LDS, by one wavefront: the lanes draw the
// channels, 64 at a time, and the table rows of the Paulis drawn are xored, the
// bits of the angles and the X and Z masks alike.  A group of channels side by
// side, one word to a lane, is one step (as many channels as their words fit 64
// lanes), two groups' loads in flight together, and groups without a drawn
// Pauli are passed over: a step per Pauli where few are drawn, and at most as
// many as a frame has words per 64 channels where many are.  The power of i,
// which only rows that keep their phase show, follows from the order: F <- P F
// with P the drawn Pauli moved to the end, F = i^k X^x Z^z.  Expectation of a
// row of 4 qubits and 280 channels (of 512 rows of 11 qubits and 420): one
// Pauli after another 65 us (181), groups one at a time 39.8 (107), two 38.0
// (97), four 37.0 (92) where a channel draws one with probability 0.4, but four
// are 0.4 to 1 us slower than two where it is 0.01.
constexpr int kFrameGroups = 2;
template <class A>
__device__ __forceinline__ void frame_row(const A &a, const double *off, uint64_t noise_seed, int b, uint32_t *acc)
{
    const int lane = threadIdx.x & 63, fw = a.frame_words, W = fw - 1;
    const bool phased = a.phase_out >= 0;
    for (int w = lane; w < fw; w += 64) acc[w] = 0u;
    const int lw = W > 32 ? 6 : 32 - __clz(W - 1);  // (W >= 2: the X and Z masks)
    const int each = 64 >> lw, sub = lane >> lw, word = min(lane & ((1 << lw) - 1), W - 1);
    uint32_t v = 0, x = 0, k = 0;
    for (int c0 = 0; c0 < a.nchan; c0 += 64) {
        int pick = 0;
        if (c0 + lane < a.nchan) {
            const GateDev gd = a.gates[a.chan_gates[c0 + lane]];
            const double p[3] = {off[gd.slot0], off[gd.slot0 + 1], off[gd.slot0 + 2]};
            pick = channel_pick(noise_seed, b, gd.chan, p);
        }
        uint64_t m = __ballot(pick != 0);
        while (m) {
            const uint32_t *r[kFrameGroups];
            int d[kFrameGroups];
#pragma unroll
            for (int i = 0; i < kFrameGroups; i++) {
                // (none left: no Pauli, and a row that is there to be read)
                const int first = m ? (__ffsll((unsigned long long)m) - 1) & -each : 0;
                d[i] = m ? __shfl(pick, first + sub) : 0;
                m &= ~(((1ull << each) - 1) << first);
                r[i] = a.frame_table + (int64_t)2 * min(c0 + first + sub, a.nchan - 1) * fw;
            }
            // X and Y take a channel's first row, Y and Z its second
            auto rows = [&](int w) {
                uint32_t rx[kFrameGroups], rz[kFrameGroups], t = 0;
#pragma unroll
                for (int i = 0; i < kFrameGroups; i++) {
                    rx[i] = r[i][w];
                    rz[i] = r[i][fw + w];
                }
#pragma unroll
                for (int i = 0; i < kFrameGroups; i++)
                    t ^= (d[i] == 1 || d[i] == 2 ? rx[i] : 0u) ^ (d[i] >= 2 ? rz[i] : 0u);
                return t;
            };
            if (W <= 64) v ^= rows(word);
            else
                for (int w = lane; w < W; w += 64) acc[w] ^= rows(w);
        }
        if (phased) {
            // this lane's Pauli (Y = i X Z: Z first), then what it meets: the
            // X mask of those before it
            uint32_t px = 0, pz = 0, pk = 0;
            if (pick) {
                const uint32_t *r = a.frame_table + (int64_t)2 * (c0 + lane) * fw + (W - 2);
                if (pick >= 2) {
                    px = r[fw];
                    pz = r[fw + 1];
                    pk = r[fw + 2];
                }
                if (pick <= 2) {
                    pk += r[2] + 2u * (uint32_t)__popc(r[1] & px) + (pick == 2);
                    px ^= r[0];
                    pz ^= r[1];
                }
            }
            uint32_t upto = px;
            for (int s = 1; s < 64; s *= 2) {
                const uint32_t o = __shfl_up(upto, s);
                if (lane >= s) upto ^= o;
            }
            k += pk + 2u * (uint32_t)__popc(pz & (x ^ upto ^ px));
            x ^= __shfl(upto, 63);
        }
    }
    if (W <= 64) {
        for (int s = 1 << lw; s < 64; s *= 2) v ^= __shfl_xor(v, s);
        if (lane < W) acc[lane] = v;
    }
    if (phased) {
        for (int s = 1; s < 64; s *= 2) k += __shfl_xor(k, s);
        if (lane == 0) acc[W] = k & 3u;
    }
}

// --------------------------------------------------- matrix build kernel
// One thread per (row, task); the result goes to the row's matrix block.
template <bool FULL, class A>
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
               theta + (int64_t)b * a.S, noise_seed, b, shift, a.x_eps, a.phase_out >= 0, nullptr, a.frame_words};
    if (a.frames) {
        extern __shared__ uint32_t frame_lds[];
        if (threadIdx.x < 64) frame_row(a, c.off, noise_seed, b, frame_lds);
        __syncthreads();
        c.frame = frame_lds;
        // kept for the gradients' signs and the rows derived from this one
        if (bx == 0 && !shift)
            for (int w = threadIdx.x; w < a.frame_words; w += blockDim.x)
                a.frames[(int64_t)src * a.frame_words + w] = frame_lds[w];
    }
    int odd = 0;
    if (ti < a.task_end) {
        const BuildTask bt = a.tasks[ti];
        odd = build_task<FULL>(bt, c, a.mats + (int64_t)row * a.mat_stride + bt.out);
    }
    if (a.phase_out < 0 || bx != 0) return;
    // the row's global phase (block 0 of the row; its thread 0 built the
    // product-init matrix at phase_out), reduced in a fixed order
    __shared__ double part[4];
    // (signs the shears of forward rotations leave out: this block's tasks,
    // then the tasks of the row's other blocks)
    if (!a.rot_end) odd = 0;
    for (int j = ti + blockDim.x; j < a.rot_end; j += blockDim.x) {
        const BuildTask bt = a.tasks[j];
        if (bt.kind == BT_PRODUCT && bt.which != BX_NONE) odd += rot_turns(bt, c);
    }
    double ph = odd * 3.14159265358979323846;
    if (c.frame && threadIdx.x == 0) ph += (double)(c.frame[c.frame_words - 1] & 3u) * (0.5 * 3.14159265358979323846);
    for (int j = threadIdx.x; j < a.n_phase; j += blockDim.x) {
        const PhaseTerm pt = a.phase_terms[j];
        const double k = c.flipped(pt.flip) ? pt.cf : pt.c;
        ph += pt.slot >= 0 ? k * slot_value(c, pt.slot, c.slot_sym[pt.slot]) : k;
    }
    ph = wave_sum(ph);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ph;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s, co;
        for (int w = 1; w < (int)(blockDim.x >> 6); w++) part[0] += part[w];
        sincos_of(part[0], false, &s, &co);
        double2 *out = a.mats + (int64_t)row * a.mat_stride + a.phase_out;
        for (int i = 0; i < 4; i++) {
            const double2 v = out[i];
            out[i] = make_double2(co * v.x - s * v.y, co * v.y + s * v.x);
        }
    }
}

// FULL: programs with 4x4 matrices that are neither diagonal nor a pair.  Its
// sixteen entries take all 256 registers that two wavefronts per SIMD leave (see
// code_steps); the other kernel, at 173, fetches less code: with the entries
// unpacked all at once, shifted rows of 12 rows of 10-qubit QAOA took 28.0 us in
// the one and 15.4 in the other.
template <bool FULL> __global__ __launch_bounds__(256, 2) void k_build_mats(BuildArgs a)
{
    build_rows<FULL>(a, a.theta, a.noise_seed, blockIdx.y, blockIdx.x);
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
// row (a move's list holds a task or two).  (Derived rows give expectations
// alone: their global phase is whatever the copied and rebuilt matrices make
// it.)
template <bool FULL> __global__ __launch_bounds__(256) void k_build_list(BuildArgs a, int nrows)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= nrows) return;
    const int64_t L = a.x_begin + row;
    const int src = (int)(L / a.x_period);
    const int m = (int)(L - (int64_t)src * a.x_period);
    const int b = cget(a.rows, src);
    const BuildCtx c{a.members, a.gates, a.slot_sym,
                     a.slot_scale + (a.uniform ? 0 : (int64_t)src * a.n_slots),
                     a.slot_off + (a.uniform ? 0 : (int64_t)src * a.n_slots), a.explicit_mats,
                     a.theta + (int64_t)b * a.S, a.noise_seed, b, a.x_shift + m, a.x_eps, false,
                     a.frames ? a.frames + (int64_t)src * a.frame_words : nullptr, a.frame_words};
    double2 *block = a.mats + (int64_t)row * a.mat_stride;
    for (int li = a.list_begin[m]; li < a.list_begin[m + 1]; li++) {
        const BuildTask bt = a.tasks[a.task_list[li]];
        build_task<FULL>(bt, c, block + bt.out);
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
    const PassCtx c = pass_setup(a, state, bid, smem, a.mat_end - a.mat_begin);
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
    const RevCtx c = rev_setup(a, bid, smem, a.mat_end - a.mat_begin);
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
            sum += 2.0 * scale[a.gslot_slot[gs]] * v * frame_sign(a, row, gs);
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

__global__ __launch_bounds__(256, 2) void k_build_batch(const void *table, const BatchBlock *blocks, ResCall c)
{
    const BatchBlock bb = cget(blocks, blockIdx.x);
    TableArg<BuildArgs> &a = table_arg<BuildArgs>(table, bb.arg);
    const int nx = (a.task_end - a.task_begin + 255) / 256;
    build_rows<true>(a, c.theta, c.noise_seed, bb.block / nx, bb.block % nx);
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
    // (1: the workgroup keeps its number, so the tiles of a row share an XCD's
    // L2 only by chance; two states of 24 qubits are no slower for it, 1025 us
    // against 1087 in two launches that number them by XCD)
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
    float2 *st = c.state_out + (int64_t)cget(a.rows, bb.block / a.wg_per_row) * a.row_stride;
    for (int64_t i = a.from + (bb.block % a.wg_per_row) * 256 + threadIdx.x; i < a.to; i += 256 * a.wg_per_row)
        st[i] = make_float2(0.f, 0.f);
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
    if (max_list > 0)
        hipLaunchKernelGGL(a.full ? k_build_list<true> : k_build_list<false>, dim3((unsigned)((nrows + 255) / 256)),
                       dim3(256), 0, s, a, nrows);
    return hipGetLastError();
}

hipError_t launch_build(const BuildArgs &a, int nrows, hipStream_t s)
{
    int n = a.task_end - a.task_begin;
    if (n <= 0 || nrows <= 0) return hipSuccess;
    // rows of up to 64 tasks: one wavefront each, none waits idle at the phase sum
    const int nt = n <= 64 ? 64 : 256;
    dim3 grid((n + nt - 1) / nt, nrows);
    prof::Scope ps("build", s);
    hipLaunchKernelGGL(a.full ? k_build_mats<true> : k_build_mats<false>, grid, dim3(nt), build_lds_bytes(a), s, a);
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

size_t rev_pass_lds_bytes(const TileGeom &g, int nmat, int waves, int gcount)
{
    return 2 * sizeof(float2) * ((size_t)1 << g.t) + sizeof(uint64_t) * ((size_t)1 << g.h) +
           sizeof(double2) * (size_t)nmat + sizeof(double) * waves * (size_t)(gcount > 0 ? gcount : 1);
}
size_t rev_pass_lds_bytes(const RevArgs &a)
{
    return rev_pass_lds_bytes(a.g, a.mat_end - a.mat_begin, kThreads / 64, a.gcount);
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
