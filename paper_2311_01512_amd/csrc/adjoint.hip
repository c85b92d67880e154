// Adjoint-method gradients of a recorded statevector circuit: parametrised
// Pauli gadgets exp(i scale theta_p P) (Sec. "Pauli gadget") of any weight
// among fixed gates and gadgets, for the energy E = <psi|H|psi> of a
// Pauli-sum observable H.
//
// Forward: psi = U_L .. U_1 psi_0, one pass per operator.  Then
// lambda = H psi and E = Re <psi|lambda>.  Backward, for k = L .. 1: if U_k
// is a parametrised gadget, dE/dtheta_p += 2 Re(i scale <lambda|P|psi>) =
// -2 scale Im <lambda|P|psi> (psi is then the state after U_k, lambda the
// back-propagated H psi); then psi <- U_k^dag psi and lambda <- U_k^dag lambda.
//
// On 9 qubits or more, with unitary gates, both directions run as tile steps
// (adjoint_tiles); otherwise one operator per pass.
#include "circuit.hpp"
#include "pauli_sum_dev.hpp"

#include <algorithm>
#include <cmath>
#include <memory>
#include <mutex>

namespace qs {

// out (+)= sum_n c_n P_n in over the terms of one launch, 256 U amplitudes per
// block (add_pauli_terms).  Bound: the gathers, which the caches serve (20
// terms on 22 qubits in complex128, 64 MiB gathered 20 times: 188 us; with
// eight operations per term and 16 terms per launch 213).
template <typename R, int U>
__global__ __launch_bounds__(256) void k_apply_pauli_sum(C2<R> *__restrict__ out, const C2<R> *__restrict__ in,
                                                          uint64_t n, PauliTerms p, int accumulate)
{
    const uint64_t first = (uint64_t)blockIdx.x * (256 * U);
    const uint32_t t = threadIdx.x;
    if (first + t >= n) return;   // states below 256 amplitudes
    double re[U], im[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        re[u] = im[u] = 0.0;
        if (accumulate) {
            const C2<R> o = out[first + 256u * u + t];
            re[u] = o.x;
            im[u] = o.y;
        }
    }
    add_pauli_terms<R, U, false>(re, im, in, first, t, p.t, 0, p.real);
    add_pauli_terms<R, U, true>(re, im, in, first, t, p.t, p.real, p.count);
#pragma unroll
    for (int u = 0; u < U; u++) out[first + 256u * u + t] = mk<R>((R)re[u], (R)im[u]);
}

// Per-block partial sums of <a|P|b> = sum_i conj(a_i) beta_j b_j, j = i ^ x,
// beta_j = (-1)^{popc(j & yz)} (the factor i^{#Y} is applied on the host).
template <typename R>
__global__ __launch_bounds__(256) void k_inner_pauli(const C2<R> *__restrict__ a, const C2<R> *__restrict__ b,
                                                      uint64_t n, uint64_t x, uint64_t yz, double *__restrict__ partials)
{
    __shared__ double s_re[4], s_im[4];
    double re = 0.0, im = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t j = i ^ x;
        const C2<R> u = a[i], v = b[j];
        const double s = (__popcll(j & yz) & 1) ? -1.0 : 1.0;
        // conj(u) v
        re += s * ((double)u.x * (double)v.x + (double)u.y * (double)v.y);
        im += s * ((double)u.x * (double)v.y - (double)u.y * (double)v.x);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o, 64);
        im += __shfl_xor(im, o, 64);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        s_re[wave] = re;
        s_im[wave] = im;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = ((s_re[0] + s_re[1]) + s_re[2]) + s_re[3];
        partials[2 * blockIdx.x + 1] = ((s_im[0] + s_im[1]) + s_im[2]) + s_im[3];
    }
}

template <typename R>
static int apply_observable(qs_qureg *lam, const qs_qureg *psi, const int *codes, const double *coeffs, int T)
{
    const uint64_t n = psi->num_amps;
    // T = 0: one launch with no terms writes zeros
    for (int b = 0; b < T || b == 0; b += kSumTerms) {
        const PauliTerms p = pauli_terms(codes, coeffs, psi->num_qubits, b, std::min(b + kSumTerms, T));
        C2<R> *out = (C2<R> *)lam->amps;
        const C2<R> *in = (const C2<R> *)psi->amps;
        if (n >= 1024)
            hipLaunchKernelGGL((k_apply_pauli_sum<R, 4>), dim3((unsigned)(n / 1024)), dim3(256), 0, lam->stream, out, in,
                               n, p, b > 0 ? 1 : 0);
        else
            hipLaunchKernelGGL((k_apply_pauli_sum<R, 1>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, lam->stream,
                               out, in, n, p, b > 0 ? 1 : 0);
        QS_LAUNCH_CHECK();
    }
    return QS_OK;
}

// <a|P|b> for the gadget string (targs, paulis), into out (re, im).
template <typename R>
static int inner_pauli(qs_qureg *a, const qs_qureg *b, const std::vector<int> &targs, const std::vector<int> &paulis,
                       double *out)
{
    uint64_t x = 0, yz = 0;
    int ny = 0;
    for (size_t k = 0; k < targs.size(); k++) {
        const uint64_t m = 1ULL << targs[k];
        if (paulis[k] == 1 || paulis[k] == 2) x |= m;
        if (paulis[k] == 2 || paulis[k] == 3) yz |= m;
        if (paulis[k] == 2) ny++;
    }
    const int blocks = (int)grid_for(a->num_amps, 256, kReduceBlocks);
    hipLaunchKernelGGL(k_inner_pauli<R>, dim3(blocks), dim3(256), 0, a->stream, (const C2<R> *)a->amps,
                       (const C2<R> *)b->amps, a->num_amps, x, yz, a->d_partials);
    QS_LAUNCH_CHECK();
    double v[2];
    int rc = finish_reduction(a, blocks, v);
    if (rc != QS_OK) return rc;
    const cd eta[4] = {cd(1, 0), cd(0, 1), cd(-1, 0), cd(0, -1)};
    const cd z = cd(v[0], v[1]) * eta[ny & 3];
    out[0] = z.real();
    out[1] = z.imag();
    return QS_OK;
}

static std::vector<cd> adjoint_of(const std::vector<cd> &M, size_t d)
{
    std::vector<cd> A(d * d);
    for (size_t r = 0; r < d; r++)
        for (size_t c = 0; c < d; c++) A[c * d + r] = std::conj(M[r * d + c]);
    return A;
}

static int apply_op(qs_qureg *q, const CircOp &op, bool adjoint)
{
    if (op.gadget) return apply_raw_gadget(q, op.targs, op.paulis, adjoint ? -op.theta : op.theta);
    if (!adjoint) return apply_raw_gate(q, op.ctrls, op.targs, op.M);
    return apply_raw_gate(q, op.ctrls, op.targs, adjoint_of(op.M, (size_t)1 << op.targs.size()));
}

// ---- the sweep as tile steps -------------------------------------------------------
//
// One operator per pass reads and writes a state for each of the sweep's
// three applications, and each gradient reads both states and waits for its
// sum.  As tile steps the forward circuit is one pass over psi per step, and
// the way back one pass over psi and lambda per step, in which the step's
// gadgets also form their gradients (k_tile_adjoint); the sums of all of them
// come back in one copy.
//
// Inside a step operators may trade places with operators they commute with.
// That leaves each gradient alone when the gates it moved across are unitary
// (<V^dag lambda|P|V^dag psi> = <lambda|P|psi> for unitary V that commutes
// with P), so circuits with other matrices keep the operator-by-operator sweep.

struct AdjointPlan {
    size_t num_ops = 0;
    int precision = -1, device = -1, num_qubits = 0;
    bool tiles = false;                 // false: the operator-by-operator sweep
    std::vector<TileStep> steps;
    std::vector<CircOp> rev;            // adjoint of every operator
    int num_grads = 0;                  // parametrised gadgets
    unsigned blocks = 0;                // grid of the steps of the way back
    // device tables of all steps (forward, then backward) and their pinned copy
    unsigned char *dev = nullptr, *host = nullptr;
    size_t bytes = 0;
    double *gpart = nullptr;            // num_grads rows of `blocks` partial sums
    double *d_out = nullptr, *h_out = nullptr;   // energy (re, im), then one sum per gradient

    AdjointPlan() = default;
    AdjointPlan(const AdjointPlan &) = delete;
    ~AdjointPlan()
    {
        release_tables();
        if (gpart) (void)hipFree(gpart);
        if (d_out) (void)hipFree(d_out);
        if (h_out) (void)hipHostFree(h_out);
    }
    void release_tables()
    {
        if (dev) (void)hipFree(dev);
        if (host) (void)hipHostFree(host);
        dev = host = nullptr;
        bytes = 0;
    }
    // At least n bytes of tables; earlier contents are lost when they grow.
    int reserve_tables(size_t n)
    {
        if (bytes >= n) return QS_OK;
        release_tables();
        if (hipMalloc(&dev, n) != hipSuccess || hipHostMalloc(&host, n, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return fail(QS_E_ALLOC, "allocation of the adjoint sweep's tables failed");
        }
        bytes = n;
        return QS_OK;
    }
};

// The plan's buffers belong to the states' device.
struct DeviceGuard {
    int before = -1;
    explicit DeviceGuard(int device)
    {
        if (hipGetDevice(&before) != hipSuccess || before == device || hipSetDevice(device) != hipSuccess) before = -1;
    }
    ~DeviceGuard()
    {
        if (before >= 0) (void)hipSetDevice(before);
    }
};

// A step's gradients share the block's LDS with its tile.
constexpr int kStepGrads = 32;
// Most doubles of gradient partials (64 MiB).
constexpr size_t kGradPartials = (size_t)1 << 23;

static bool is_unitary(const CircOp &op, double tol)
{
    const size_t d = (size_t)1 << op.targs.size();
    for (size_t r = 0; r < d; r++)
        for (size_t c = 0; c <= r; c++) {
            cd z = r == c ? cd(-1, 0) : cd(0, 0);
            for (size_t k = 0; k < d; k++) z += op.M[r * d + k] * std::conj(op.M[c * d + k]);
            if (!(std::abs(z) <= tol)) return false;
        }
    return true;
}

// Tiles of 2^12 (complex64) or 2^11 (complex128) amplitudes: both states of a
// tile take 32 KiB of LDS in turn.
static int adjoint_tile_dim(int precision, int num_qubits)
{
    return std::min({num_qubits, precision == QS_C64 ? 12 : 11, tile_dim_limit(precision)});
}

static int build_adjoint_plan(AdjointPlan &pl, const qs_circuit *c, const qs_qureg *psi)
{
    pl.num_ops = c->ops.size();
    pl.precision = psi->precision;
    pl.device = psi->device;
    pl.num_qubits = c->num_qubits;
    // the gradients' wave sums need whole wavefronts: tiles of 2^9 or more
    const int T = adjoint_tile_dim(pl.precision, c->num_qubits);
    if (T < kRegBits + 6) return QS_OK;
    // rounding of a matrix given in the state's precision is let through
    const double tol = pl.precision == QS_C64 ? 1e-6 : 1e-13;
    for (const auto &op : c->ops)
        if (!op.gadget && !is_unitary(op, tol)) return QS_OK;
    pl.steps = group_tile_steps(c->ops, c->num_qubits, T, pl.precision, -1, kStepGrads);
    pl.rev = c->ops;
    for (auto &op : pl.rev) {
        if (!op.gadget) op.M = adjoint_of(op.M, (size_t)1 << op.targs.size());
        else if (op.param >= 0) pl.num_grads++;
    }
    const uint64_t tiles = 1ULL << (c->num_qubits - T);
    pl.blocks = (unsigned)std::min<uint64_t>(tiles, 2048);
    while (pl.blocks > 256 && (size_t)pl.blocks * pl.num_grads > kGradPartials) pl.blocks /= 2;
    const size_t out = sizeof(double) * (2 + (size_t)pl.num_grads);
    if (hipMalloc(&pl.gpart, sizeof(double) * std::max<size_t>(1, (size_t)pl.blocks * pl.num_grads)) != hipSuccess ||
        hipMalloc(&pl.d_out, out) != hipSuccess || hipHostMalloc(&pl.h_out, out, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return fail(QS_E_ALLOC, "allocation of the adjoint sweep's sums failed");
    }
    pl.tiles = true;
    return QS_OK;
}

// Encodes one direction's steps, in application order, with the angles of
// `ops` (the circuit's operators, or their adjoints last first).
static std::vector<Pass> encode_direction(const AdjointPlan &pl, const std::vector<CircOp> &ops, bool back)
{
    std::vector<Pass> out(pl.steps.size());
    const bool mfma = pl.precision == QS_C64;
    for (size_t k = 0; k < pl.steps.size(); k++) {
        const TileStep &st = pl.steps[back ? pl.steps.size() - 1 - k : k];
        if (st.single >= 0) continue;
        std::vector<const CircOp *> members;
        for (int j : st.members) members.push_back(&ops[j]);
        if (back) std::reverse(members.begin(), members.end());
        encode_step(out[k], st.span, members, mfma, back);
    }
    return out;
}

// Gives the passes their places in the plan's tables from `offset` on;
// returns the end.
static size_t place_tables(const AdjointPlan &pl, std::vector<Pass> &passes, size_t offset)
{
    for (Pass &p : passes) {
        if (!p.tile) continue;
        p.dev_offset = offset;
        offset += (tile_pass_bytes(p, pl.precision) + 255) & ~size_t(255);
    }
    return offset;
}

// Copies the passes' tables to the device, ordered on the stream.
static int upload_tables(AdjointPlan &pl, const std::vector<Pass> &passes, size_t begin, size_t end, hipStream_t stream)
{
    for (const Pass &p : passes)
        if (p.tile) pack_tile_pass(p, pl.precision, pl.host + p.dev_offset);
    if (end > begin) QS_HIP(hipMemcpyAsync(pl.dev + begin, pl.host + begin, end - begin, hipMemcpyHostToDevice, stream));
    return QS_OK;
}

template <typename R>
static int adjoint_tiles(AdjointPlan &pl, const qs_circuit *c, qs_qureg *psi, qs_qureg *lam, const int *codes,
                         const double *coeffs, int T, int num_params, double *energy, double *grads)
{
    for (size_t k = 0; k < c->ops.size(); k++)
        if (c->ops[k].gadget) pl.rev[k].theta = -c->ops[k].theta;
    std::vector<Pass> fwd = encode_direction(pl, c->ops, false);
    const size_t mid = place_tables(pl, fwd, 0);
    // room for the way back as well: its tables hold the same operators (and
    // at most one scaling operator more per step)
    int rc = pl.reserve_tables(2 * mid + 1024 * pl.steps.size() + 4096);
    if (rc == QS_OK) rc = upload_tables(pl, fwd, 0, mid, psi->stream);
    if (rc != QS_OK) return rc;
    const size_t S = pl.steps.size();
    for (size_t k = 0; k < S; k++) {
        const TileStep &st = pl.steps[k];
        rc = st.single >= 0 ? apply_op(psi, c->ops[st.single], false) : launch_tile_pass(psi, fwd[k], pl.dev + fwd[k].dev_offset);
        if (rc != QS_OK) return rc;
    }
    rc = apply_observable<R>(lam, psi, codes, coeffs, T);
    if (rc == QS_OK) rc = queue_inner_product(psi, lam, pl.d_out);
    if (rc != QS_OK) return rc;
    // encoded while the device runs the above
    std::vector<Pass> back = encode_direction(pl, pl.rev, true);
    const size_t end = place_tables(pl, back, mid);
    if (end > pl.bytes) {
        // fused differently, they can be larger: wait for the forward steps
        QS_HIP(hipStreamSynchronize(psi->stream));
        rc = pl.reserve_tables(end);
    }
    if (rc == QS_OK) rc = upload_tables(pl, back, mid, end, psi->stream);
    if (rc != QS_OK) return rc;
    size_t row = 0;
    for (size_t k = 0; k < S; k++) {
        const TileStep &st = pl.steps[S - 1 - k];
        if (st.single >= 0) {
            rc = apply_op(psi, c->ops[st.single], true);
            if (rc == QS_OK) rc = apply_op(lam, c->ops[st.single], true);
        } else {
            rc = launch_adjoint_pass(psi, lam, back[k], pl.dev + back[k].dev_offset, pl.gpart + row * pl.blocks, pl.blocks);
            row += back[k].grads.size();
        }
        if (rc != QS_OK) return rc;
    }
    rc = queue_row_sums(psi->stream, pl.gpart, (int)row, (int)pl.blocks, pl.d_out + 2);
    if (rc != QS_OK) return rc;
    QS_HIP(hipMemcpyAsync(pl.h_out, pl.d_out, sizeof(double) * (2 + row), hipMemcpyDeviceToHost, psi->stream));
    QS_HIP(hipStreamSynchronize(psi->stream));
    *energy = pl.h_out[0];
    for (int p = 0; p < num_params; p++) grads[p] = 0.0;
    const double *sum = pl.h_out + 2;
    for (const Pass &p : back)
        for (const GradRef &g : p.grads) grads[g.param] += g.weight * *sum++;
    return QS_OK;
}

template <typename R>
static int adjoint_sweep(qs_circuit *c, qs_qureg *psi, qs_qureg *lam, const int *codes, const double *coeffs,
                         int T, int num_params, double *energy, double *grads)
{
    const DeviceGuard guard(psi->device);
    std::shared_ptr<AdjointPlan> pl;
    {
        std::lock_guard<std::mutex> lock(c->adjoint_mu);
        pl.swap(c->adjoint);
    }
    int rc = QS_OK;
    // operators are only ever appended: the same count, the same structure
    if (!pl || pl->num_ops != c->ops.size() || pl->precision != psi->precision || pl->device != psi->device) {
        pl = std::make_shared<AdjointPlan>();
        rc = build_adjoint_plan(*pl, c, psi);
        if (rc != QS_OK) return rc;
    }
    if (pl->tiles) {
        rc = adjoint_tiles<R>(*pl, c, psi, lam, codes, coeffs, T, num_params, energy, grads);
        if (rc != QS_OK) {
            (void)hipStreamSynchronize(psi->stream);   // queued steps read the plan's tables
            return rc;
        }
    }
    {
        std::lock_guard<std::mutex> lock(c->adjoint_mu);
        c->adjoint = pl;
    }
    if (pl->tiles) return QS_OK;
    for (int p = 0; p < num_params; p++) grads[p] = 0.0;
    for (const auto &op : c->ops) {
        rc = apply_op(psi, op, false);
        if (rc != QS_OK) return rc;
    }
    rc = apply_observable<R>(lam, psi, codes, coeffs, T);
    if (rc != QS_OK) return rc;
    double re = 0.0, im = 0.0;
    rc = qs_calc_inner_product(psi, lam, &re, &im);
    if (rc != QS_OK) return rc;
    *energy = re;
    for (size_t k = c->ops.size(); k-- > 0;) {
        const CircOp &op = c->ops[k];
        if (op.gadget && op.param >= 0) {
            double z[2];
            rc = inner_pauli<R>(lam, psi, op.targs, op.paulis, z);
            if (rc != QS_OK) return rc;
            grads[op.param] += -2.0 * op.scale * z[1];
        }
        rc = apply_op(psi, op, true);
        if (rc == QS_OK) rc = apply_op(lam, op, true);
        if (rc != QS_OK) return rc;
    }
    return QS_OK;
}

}  // namespace qs

using namespace qs;

extern "C" {

int qs_circuit_add_param_gadget(qs_circuit *c, const int *targs, const int *paulis, int num_targs, int param,
                                double scale)
{
    if (!c) return fail(QS_E_ARG, "null circuit");
    if (c->is_density) return fail(QS_E_PRECOND, "parametrised gadgets belong to statevector circuits");
    if (param < 0) return fail(QS_E_ARG, "negative parameter index");
    int rc = qs_circuit_add_pauli_gadget(c, targs, paulis, num_targs, 0.0);
    if (rc != QS_OK) return rc;
    c->ops.back().param = param;
    c->ops.back().scale = scale;
    return QS_OK;
}

int qs_circuit_set_params(qs_circuit *c, const double *params, int num_params)
{
    if (!c) return fail(QS_E_ARG, "null circuit");
    if (num_params < 0 || (num_params > 0 && !params)) return fail(QS_E_ARG, "bad parameter vector");
    for (const auto &op : c->ops)
        if (op.param >= num_params) return fail(QS_E_ARG, "parameter index beyond the vector");
    for (auto &op : c->ops)
        if (op.param >= 0) op.theta = op.scale * params[op.param];
    // compiled passes hold the old angles
    release_specialized(c);
    c->compiled = false;
    return QS_OK;
}

int qs_circuit_adjoint_gradient(qs_circuit *c, qs_qureg *psi, qs_qureg *lam, const int *paulis,
                                const double *coeffs, int num_terms, int num_params, double *energy, double *grads)
{
    if (!c || !psi || !lam || !energy || (num_params > 0 && !grads)) return fail(QS_E_ARG, "null argument");
    if (num_terms < 0 || (num_terms > 0 && (!paulis || !coeffs))) return fail(QS_E_ARG, "bad observable");
    if (c->is_density || psi->is_density || lam->is_density)
        return fail(QS_E_PRECOND, "adjoint gradients of statevector circuits");
    if (psi->num_qubits != c->num_qubits || lam->num_qubits != c->num_qubits)
        return fail(QS_E_ARG, "qubit counts differ");
    if (psi->precision != lam->precision) return fail(QS_E_TYPE, "precisions differ");
    if (psi->amps == lam->amps) return fail(QS_E_ARG, "psi and lambda must not alias");
    if (psi->stream != lam->stream) return fail(QS_E_ARG, "psi and lambda must share a stream");
    for (int i = 0; i < num_terms * c->num_qubits; i++)
        if (paulis[i] < 0 || paulis[i] > 3) return fail(QS_E_ARG, "Pauli codes are 0..3");
    for (const auto &op : c->ops)
        if (op.param >= num_params) return fail(QS_E_ARG, "parameter index beyond num_params");
    return psi->precision == QS_C64
               ? adjoint_sweep<float>(c, psi, lam, paulis, coeffs, num_terms, num_params, energy, grads)
               : adjoint_sweep<double>(c, psi, lam, paulis, coeffs, num_terms, num_params, energy, grads);
}

}  // extern "C"
