// jit.cpp -- per-plan code generation of the fused pass kernels.
//
// The interpreter kernels in qsv.hip read the pass/stage/op tables at run time;
// every op then ends in a data-dependent branch, and the compiler has to copy
// all register amplitudes back into place after it. Here the same tables are
// turned into HIP source instead: one straight-line kernel per pass, with the
// tile layout, the register position of every gate, the sign masks of CZ
// groups and the gradient slots as constants. Only the gate matrices (which
// depend on the weights and inputs of a call) are read from memory. The
// source is compiled for the device's architecture once per plan and device:
// by the ROCm clang driver in parallel child processes (one per kernel) when it
// is installed, else by hipRTC (which serialises compilations in a process).
//
// Every generated kernel applies the same ops in the same order as the
// matching table-driven kernel; only float32 contraction and the order of the
// per-thread gradient sums differ.
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>
#include <fcntl.h>
#include <spawn.h>
#include <sys/stat.h>
#include <sys/wait.h>
#include <unistd.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <sstream>
#include <string>
#include <thread>
#include <vector>

#include "jit.hpp"

namespace qsv {
namespace {

std::string I(long long v) { return std::to_string(v); }

std::string hex(unsigned v) {
    char b[16];
    std::snprintf(b, sizeof b, "0x%xu", v);
    return b;
}

// Expression placing bit i of `var` at position pos[i] (runs of consecutive
// positions are moved with one shift and mask).
std::string scatter(const std::string& var, const std::vector<int>& pos) {
    std::string s;
    const int n = (int)pos.size();
    int i = 0;
    while (i < n) {
        int j = i;
        while (j + 1 < n && pos[j + 1] == pos[j] + 1) ++j;
        const int len = j - i + 1;
        std::string term = i ? "(" + var + " >> " + I(i) + ")" : var;
        term = "(" + term + " & " + hex((1u << len) - 1) + ")";
        if (pos[i]) term = "(" + term + " << " + I(pos[i]) + ")";
        s += (s.empty() ? "" : " | ") + term;
        i = j + 1;
    }
    return s.empty() ? "0" : s;
}

int swz_host(int l) { return l ^ (((l >> 5) ^ (l >> 10)) & 31); }

// Where a tile's local bits live: four in the register index, the others in
// the thread index (the six lane bits first, then the wave bits).
struct Layout {
    int reg[kRegBits];
    std::vector<int> nonreg;  // local bit of thread-index bit i
};

constexpr int kLaneBits = 6;

// `wave`: mask of the local bits on the wave index; lane and wave bits ascend.
Layout make_layout(int m, const int* reg, unsigned wave) {
    Layout L;
    for (int p = 0; p < kRegBits; ++p) L.reg[p] = reg[p];
    for (int w = 0; w < 2; ++w)
        for (int j = 0; j < m; ++j)
            if (std::find(reg, reg + kRegBits, j) == reg + kRegBits && (int)(wave >> j & 1) == w) L.nonreg.push_back(j);
    return L;
}

// mask of the top local bits outside `reg`, as many as there are wave bits
unsigned top_wave_bits(int m, const int* reg) {
    unsigned w = 0;
    for (int j = m - 1, n = std::max(0, m - kRegBits - kLaneBits); n > 0; --j)
        if (std::find(reg, reg + kRegBits, j) == reg + kRegBits) {
            w |= 1u << j;
            --n;
        }
    return w;
}

unsigned wave_bits(const Layout& L) {
    unsigned w = 0;
    for (size_t i = kLaneBits; i < L.nonreg.size(); ++i) w |= 1u << L.nonreg[i];
    return w;
}

bool same(const Layout& a, const Layout& b) {
    return std::equal(a.reg, a.reg + kRegBits, b.reg) && a.nonreg == b.nonreg;
}

class Gen {
public:
    Gen(const qsv_plan_t* p) : p_(p) {}

    std::string prelude() const {
        return R"(
typedef float2 f2;
typedef float qsv_v4f __attribute__((ext_vector_type(4)));
typedef __UINTPTR_TYPE__ qsv_uptr;  // pointer-sized integer without any header
// Raw buffer accesses: per-thread byte offset plus a scalar one, within `bytes` of p.
typedef unsigned qsv_u2 __attribute__((ext_vector_type(2)));
typedef unsigned qsv_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t qsv_buf(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ f2 qsv_ld2(__amdgpu_buffer_rsrc_t b, int off, int c) {
    const qsv_u2 v = __builtin_amdgcn_raw_buffer_load_b64(b, off, c, 0);
    return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}
// NT: non-temporal
template <int NT>
__device__ __forceinline__ float4 qsv_ld4(__amdgpu_buffer_rsrc_t b, int off, int c) {
    const qsv_u4 v = __builtin_amdgcn_raw_buffer_load_b128(b, off, c, NT ? 2 : 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ void qsv_st2(f2 a, __amdgpu_buffer_rsrc_t b, int off, int c) {
    __builtin_amdgcn_raw_buffer_store_b64(qsv_u2{__float_as_uint(a.x), __float_as_uint(a.y)}, b, off, c, 0);
}
template <int NT>
__device__ __forceinline__ void qsv_st4(float4 a, __amdgpu_buffer_rsrc_t b, int off, int c) {
    __builtin_amdgcn_raw_buffer_store_b128(
        qsv_u4{__float_as_uint(a.x), __float_as_uint(a.y), __float_as_uint(a.z), __float_as_uint(a.w)}, b, off, c, NT ? 2 : 0);
}
// float64 wavefront sum by DPP lane moves: pairs, quads, half rows, rows, then
// row 0 -> 1, 2 -> 3 and rows 0-1 -> 2-3 broadcasts; lane 63 holds the total.
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double qsv_dpp(double v) {
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWMASK, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWMASK, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double qsv_wave_sum(double v) {
    v += qsv_dpp<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += qsv_dpp<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    v += qsv_dpp<0x141, 0xF>(v);   // row_half_mirror
    v += qsv_dpp<0x140, 0xF>(v);   // row_mirror
    v += qsv_dpp<0x142, 0xA>(v);   // row_bcast:15 into rows 1, 3
    v += qsv_dpp<0x143, 0xC>(v);   // row_bcast:31 into rows 2, 3
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)x, 63), hi = __builtin_amdgcn_readlane((int)(x >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// float32 sum over the 16 lanes of a DPP row (pairs, quads, half rows, rows);
// every lane of the row ends with the row's total.
template <int CTRL>
__device__ __forceinline__ float qsv_dppf(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float qsv_row_sum(float v) {
    v += qsv_dppf<0xB1>(v);
    v += qsv_dppf<0x4E>(v);
    v += qsv_dppf<0x141>(v);
    v += qsv_dppf<0x140>(v);
    return v;
}
// Row sums of four values at once: the four lanes of bank 0, 1, 2, 3 of a row
// (lane bits 2 and 3) end with the row's total of a, b, c, d. A bank mask keeps
// one value in half of the banks while the other half takes the next value, so
// four sums take 8 additions instead of 16 and one store instead of four. Two
// wait states lie between a write and a DPP read of it.
__device__ __forceinline__ float qsv_row_sum4(float a, float b, float c, float d) {
    __asm__ volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %2, %2 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %3, %3 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
        : "+&v"(a), "+&v"(b) : "v"(c), "v"(d));
    return a;
}
// LDS accesses of one wave to its own part of the array complete in order;
// this keeps the compiler from moving them across.
__device__ __forceinline__ void qsv_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// gradient of a gate inside a 1-qubit chain: Im<l|V P V^dagger|psi> from the
// chain's components cx, cy, cz = Im<l|X|psi>, Im<l|Y|psi>, Im<l|Z|psi>, with
// V the later gates' product (row-major 2x2) and P = X, Y, Z for axis 0, 1, 2;
// V P V^dagger = H00 Z + Re(H01) X - Im(H01) Y
__device__ double qsv_chain_grad(const float* V, int axis, double cx, double cy, double cz) {
    const double ar = V[0], ai = V[1], br = V[2], bi = V[3], cr = V[4], ci = V[5], dr = V[6], di = V[7];
    double h00, hr, hi;
    if (axis == 2) {
        h00 = ar * ar + ai * ai - br * br - bi * bi;
        hr = (ar * cr + ai * ci) - (br * dr + bi * di);
        hi = (ai * cr - ar * ci) - (bi * dr - br * di);
    } else if (axis == 0) {
        h00 = 2.0 * (ar * br + ai * bi);
        hr = (br * cr + bi * ci) + (ar * dr + ai * di);
        hi = (bi * cr - br * ci) + (ai * dr - ar * di);
    } else {
        h00 = -2.0 * (bi * ar - br * ai);
        hr = -((bi * cr - br * ci) - (ai * dr - ar * di));
        hi = (br * cr + bi * ci) - (ar * dr + ai * di);
    }
    return h00 * cz + hr * cx - hi * cy;
}
__device__ __forceinline__ f2 qsv_flip(f2 a, unsigned w) {
    const unsigned s = w & 0x80000000u;
    return make_float2(__uint_as_float(__float_as_uint(a.x) ^ s), __uint_as_float(__float_as_uint(a.y) ^ s));
}
)";
    }

    std::string kernel(int which, int i, std::string& name) {
        const DPass& ps = which == 0 ? p_->fwd_pass[i] : p_->bwd_pass[i];
        name = std::string(which == 0 ? "qsv_f" : "qsv_b") + I(i);
        o_.str("");
        bwd_ = which == 1;
        last_fwd_ = which == 0 && i + 1 == (int)p_->fwd_pass.size();
        ps_ = &ps;
        m_ = ps.m;
        W_ = p_->W;
        T_ = 1 << (m_ - kRegBits);
        threads_ = std::max(64, T_);
        guard_ = threads_ > T_;
        arrays_ = bwd_ ? std::vector<std::string>{"ps", "lm"} : std::vector<std::string>{"a"};
        emit_kernel(name);
        return o_.str();
    }

private:
    const qsv_plan_t* p_;
    const DPass* ps_ = nullptr;
    const Layout* lay_ = nullptr;  // register layout of the ops being emitted
    std::ostringstream o_;
    bool bwd_ = false, guard_ = false, last_fwd_ = false;
    bool lds_own_ = false;  // the last exchange stayed within waves (no barrier since)
    std::string name_;
    int m_ = 0, W_ = 0, T_ = 0, threads_ = 0;
    std::vector<std::string> arrays_;

    std::string act(const std::string& body) const { return guard_ ? "if (act) { " + body + " }" : body; }

    // Matrix-core path for a generic 2x2: only where every lane of the wave
    // executes it (matrix instructions run on all lanes regardless of the
    // execution mask), i.e. not under a control outside the registers.
    // opts.mfma bits: 1 forward kernels, 2 backward psi array, 4 backward lambda array.
    bool use_mfma(const DOp& op) const {
        return (p_->opts.mfma & (bwd_ ? 6 : 1)) && op.kind == OP_U2 && op.ctl < kCtlNonReg &&
               op.ctl2 < kCtlNonReg;
    }
    bool mfma_array(const std::string& A) const {
        if (!bwd_) return p_->opts.mfma & 1;
        return p_->opts.mfma & (A == "ps" ? 2 : 4);
    }

    int lq(int j) const { return ps_->lq[j]; }

    // Register bits of the layout a pass loads and stores in: the top three
    // tile bits, plus tile bit 0 when it is amplitude bit 0 (then a register
    // pair k, k + 1 holds two adjacent amplitudes), else the fourth-highest.
    std::array<int, kRegBits> nat_reg() const {
        return {lq(0) == 0 ? 0 : m_ - 4, m_ - 3, m_ - 2, m_ - 1};
    }

    Layout nat_layout() const { return make_layout(m_, nat_reg().data(), top_wave_bits(m_, nat_reg().data())); }

    // global offset of register k (within the sample) in layout L
    int gR(const Layout& L, int k) const {
        int v = 0;
        for (int p = 0; p < kRegBits; ++p)
            if (k >> p & 1) v |= 1 << lq(L.reg[p]);
        return v;
    }
    int lR(const Layout& L, int k) const {
        int v = 0;
        for (int p = 0; p < kRegBits; ++p)
            if (k >> p & 1) v |= 1 << L.reg[p];
        return v;
    }
    std::string gT_expr(const Layout& L) const {
        std::vector<int> pos;
        for (int j : L.nonreg) pos.push_back(lq(j));
        return "base | " + scatter("t", pos);
    }
    std::string lT_expr(const Layout& L) const { return scatter("t", L.nonreg); }

    // Re-lays the tile out through LDS. When both layouts keep the same local
    // bits on the wave index, every wave reads only what it wrote itself and no
    // barrier is needed; choose_waves() picks those bits so that this is the
    // common case. Byte offsets: an XOR per access and nothing else (a shift
    // more per access before). With these, the shared Z products, the merged row
    // sums and the buffer accesses, 20-qubit ladder, batch 64: 7.6 -> 7.2 ms per
    // step (longest pass 18,500 -> 17,400 vector instructions); 16-qubit ring,
    // batch 256: 1.89 -> 1.85 ms; 21-qubit ring forward, batch 7: 775 -> 750 us.
    void emit_exchange(const Layout& from, const Layout& to) {
        const bool own = wave_bits(from) == wave_bits(to);
        const char* sync = own ? "qsv_wave_sync();" : "__syncthreads();";
        // waves may still be reading their own parts
        if (!own && lds_own_) o_ << "  __syncthreads();\n";
        lds_own_ = own;
        // The empty asm statements make each exchange compute its LDS
        // addresses afresh: otherwise the compiler keeps the addresses of
        // every layout alive across the whole kernel (tens of registers).
        o_ << "  {\n    int l0_ = " << lT_expr(from) << ";\n"
           << "    __asm__ volatile(\"\" : \"+v\"(l0_));\n"
           << "    const int s0_ = (l0_ ^ (((l0_ >> 5) ^ (l0_ >> 10)) & 31)) << 3;\n"
           << "    int l1_ = " << lT_expr(to) << ";\n"
           << "    __asm__ volatile(\"\" : \"+v\"(l1_));\n"
           << "    const int s1_ = (l1_ ^ (((l1_ >> 5) ^ (l1_ >> 10)) & 31)) << 3;\n"
           << "    char* const lb_ = (char*)lds;\n";
        for (size_t ai = 0; ai < arrays_.size(); ++ai) {
            const std::string& A = arrays_[ai];
            std::string w, r;
            for (int k = 0; k < kRegs; ++k) {
                w += "*(f2*)(lb_ + (s0_ ^ " + I(swz_host(lR(from, k)) * 8) + ")) = " + A + "[" + I(k) + "]; ";
                r += A + "[" + I(k) + "] = *(const f2*)(lb_ + (s1_ ^ " + I(swz_host(lR(to, k)) * 8) + ")); ";
            }
            if (ai > 0) o_ << "    " << sync << "\n";
            o_ << "    " << act(w) << "\n    " << sync << "\n    " << act(r) << "\n";
        }
        o_ << "    " << sync << "\n  }\n";
        o_ << "  gT = " << gT_expr(to) << ";\n";
    }

    // Wave bits of every stage's layout, given the load / store layout's: as few
    // changes from one layout to the next as possible (each costs barriers),
    // the topmost bits among equals.
    std::vector<Layout> choose_waves(const Layout& nat, bool write_back) const {
        const int nw = std::max(0, m_ - kRegBits - kLaneBits), ns = ps_->n_stages;
        std::vector<std::vector<unsigned>> opt(ns);
        std::vector<std::vector<int>> cost(ns), from(ns);
        for (int s = 0; s < ns; ++s) {
            const int* reg = p_->stages[ps_->stage0 + s].reg;
            unsigned rm = 0;
            for (int p = 0; p < kRegBits; ++p) rm |= 1u << reg[p];
            for (unsigned w = 0; w < (1u << m_); ++w)
                if (__builtin_popcount(w) == nw && !(w & rm)) opt[s].push_back(w);
            std::reverse(opt[s].begin(), opt[s].end());
            for (unsigned w : opt[s]) {
                int best = 1 << 30, at = 0;
                if (s == 0) {
                    best = w == wave_bits(nat) ? 0 : 1;
                } else {
                    const bool same_reg = std::equal(reg, reg + kRegBits, p_->stages[ps_->stage0 + s - 1].reg);
                    for (size_t i = 0; i < opt[s - 1].size(); ++i) {
                        // same registers: no exchange at all, unless the wave bits changed
                        const int c = cost[s - 1][i] + (w == opt[s - 1][i] ? 0 : same_reg ? 3 : 1);
                        if (c < best) best = c, at = (int)i;
                    }
                }
                if (s == ns - 1 && write_back) best += w == wave_bits(nat) ? 0 : 1;
                cost[s].push_back(best);
                from[s].push_back(at);
            }
        }
        std::vector<Layout> out(ns);
        int i = ns ? (int)(std::min_element(cost[ns - 1].begin(), cost[ns - 1].end()) - cost[ns - 1].begin()) : 0;
        for (int s = ns - 1; s >= 0; --s) {
            out[s] = make_layout(m_, p_->stages[ps_->stage0 + s].reg, opt[s][i]);
            i = from[s][i];
        }
        return out;
    }

    std::string mat_ptr(int mat) const {
        if (mat >= 0) return "mats + " + I(8LL * mat);
        return "mp + " + I(8LL * (-mat - 1));
    }

    static std::string rk(const std::string& A, int k) { return A + "[" + I(k) + "]"; }

    // Matrix-core operands of a pass. A matrix instruction can take its A operand
    // from one block of four lanes for all 16 (cbsz 4, abid = the block), so one
    // register holds the four columns of four gates: lane l has gate l >> 4, column
    // (l >> 2) & 3, row l & 3 of the real 4x4 form of [[u00, u01], [u10, u11]] acting on
    // (x.re, x.im, y.re, y.im). One load and one sign flip (row re, column im) per
    // four consecutive matrix slots; the next group's load is issued when a group is
    // first used. Selecting the columns from scalars took 16 vector instructions per
    // gate, and a matrix instruction and a vector instruction of one SIMD do not
    // overlap (20-qubit ladder, longest forward pass: 2,624 x 8 + 2,336 x 4 cycles a
    // wave, 85% of the time it took). With this and the signs below, forward of the
    // 20-qubit ladder, batch 64: 2.40 -> 2.07 ms; 12 qubits, batch 500: 43 -> 33 us.
    struct AGroup { int mat; bool ps; };
    std::vector<AGroup> agroups_;
    std::vector<int> agroup_of_, ablock_of_;  // per op of the pass, from its first op
    int aissued_ = 0, aop0_ = 0;
    void plan_a_operands() {
        agroups_.clear();
        aissued_ = 0;
        if (!ps_->n_stages) return;
        aop0_ = p_->stages[ps_->stage0].op0;
        const int n = p_->stages[ps_->stage0 + ps_->n_stages - 1].op1 - aop0_;
        agroup_of_.assign(n, -1);
        ablock_of_.assign(n, 0);
        int open[2] = {-1, -1};  // open group of shared, per-sample matrices
        for (int i = 0; i < n; ++i) {
            const DOp& op = p_->ops[aop0_ + i];
            if (!use_mfma(op)) continue;
            const bool ps = op.mat < 0;
            const int slot = ps ? -op.mat - 1 : op.mat;
            int& g = open[ps];
            if (g < 0 || slot < agroups_[g].mat || slot >= agroups_[g].mat + 4) {
                g = (int)agroups_.size();
                agroups_.push_back({slot, ps});
            }
            agroup_of_[i] = g;
            ablock_of_[i] = 4 * (slot - agroups_[g].mat);
        }
        if (agroups_.empty()) return;
        // byte offset of the lane's entry within its group and its sign; slots past
        // the last matrix lie past the buffer's end and read as 0
        o_ << "  const int ao_ = ((t & 0x30) << 1) | ((t & 2) << 3) | (t & 8) | (((t ^ (t >> 2)) & 1) << 2);\n"
           << "  const unsigned as_ = (unsigned)((t >> 2) & ~t & 1) << 31;\n"
           << "  const __amdgpu_buffer_rsrc_t mb_ = qsv_buf(mats, (unsigned)n_shared * 32u), "
              "pb_ = qsv_buf(mp, (unsigned)n_ps * 32u); (void)mb_; (void)pb_;\n";
        issue_a_group();
    }
    void issue_a_group() {
        if (aissued_ >= (int)agroups_.size()) return;
        const AGroup& g = agroups_[aissued_];
        o_ << "  const unsigned am" << aissued_ << "_ = __builtin_amdgcn_raw_buffer_load_b32(" << (g.ps ? "pb_" : "mb_")
           << ", ao_, " << 32 * g.mat << ", 0);\n";
        ++aissued_;
    }
    // before an op: loads one group ahead of the first use of its own
    void need_a_group(int op) {
        const int g = agroups_.empty() ? -1 : agroup_of_[op - aop0_];
        while (g >= 0 && aissued_ < std::min(g + 2, (int)agroups_.size())) issue_a_group();
    }

    void emit_matrix(const DOp& op) {
        o_ << "    const float* M_ = " << mat_ptr(op.mat) << ";\n";
        switch (op.kind) {
        case OP_U2:
            if (use_mfma(op)) {
                bool valu_too = false;
                for (const std::string& A : arrays_) valu_too |= !mfma_array(A);
                if (!valu_too) break;
                o_ << "    const float m0r = M_[0], m0i = M_[1], m1r = M_[2], m1i = M_[3], "
                      "m2r = M_[4], m2i = M_[5], m3r = M_[6], m3i = M_[7];\n";
            } else {
                o_ << "    const float m0r = M_[0], m0i = M_[1], m1r = M_[2], m1i = M_[3], "
                      "m2r = M_[4], m2i = M_[5], m3r = M_[6], m3i = M_[7];\n";
            }
            break;
        case OP_REAL:
            o_ << "    const float m0r = M_[0], m1r = M_[2], m2r = M_[4], m3r = M_[6];\n";
            break;
        case OP_RXL:
            o_ << "    const float al = M_[0], be = M_[3];\n";
            break;
        case OP_DIAG:
            o_ << "    const float m0r = M_[0], m0i = M_[1], m3r = M_[6], m3i = M_[7];\n";
            break;
        default: break;
        }
    }

    // pairs (k, k | 1<<pos) of an op on register position `pos`; with a control
    // on a register position, only pairs where that bit is 1.
    // register k satisfies the op's controls that sit on register positions
    static bool reg_ok(const DOp& op, int k) {
        for (int c : {op.ctl, op.ctl2})
            if (c >= 0 && c < kCtlNonReg && !(k >> c & 1)) return false;
        return true;
    }
    // Whether a control outside the registers sits on an index bit fed by one
    // of the six lane bits of the thread index (the condition then differs
    // between the lanes of a wave). Other controls are uniform over a wave:
    // their bit lies outside the tile or comes from the wave index.
    bool lane_ctl(const DOp& op) const {
        for (int x : {op.ctl, op.ctl2}) {
            if (x < kCtlNonReg) continue;
            for (size_t i = 0; i < lay_->nonreg.size() && i < 6; ++i)
                if (lq(lay_->nonreg[i]) == (x & 0xFF)) return true;
        }
        return false;
    }
    // run-time condition of the op's controls outside the registers ("" if
    // none); a wave-uniform one is read from the first lane, so the compiler
    // branches on a scalar and skips the op for waves where it is false
    std::string nonreg_cond(const DOp& op) const {
        std::string c;
        for (int x : {op.ctl, op.ctl2})
            if (x >= kCtlNonReg) c += std::string(c.empty() ? "" : " && ") + "((gT >> " + I(x & 0xFF) + ") & 1)";
        if (c.empty() || lane_ctl(op)) return c;
        return "__builtin_amdgcn_readfirstlane((int)(" + c + "))";
    }
    std::vector<int> pairs(const DOp& op) const {
        std::vector<int> v;
        for (int k = 0; k < kRegs; ++k) {
            if (k >> op.pos & 1) continue;
            if (!reg_ok(op, k)) continue;
            v.push_back(k);
        }
        return v;
    }

    // Matrix-core form of a generic 2x2 over every pair of every state array:
    // 16 blocks of 4 lanes; a lane supplies its own pair (B operand) and receives
    // its pair's four outputs, the gate's real 4x4 form (A operand) comes from
    // plan_a_operands(). The four rank-1 steps are issued step by step across all
    // pairs, so consecutive matrix instructions are independent.
    void emit_pairs_mfma(const DOp& op) {
        struct Pair { std::string first, second, a0, a1; };
        std::vector<Pair> xy;
        bool neg = false;
        auto col = [&](int k) {
            const bool n = neg_ >> k & 1;
            neg |= n;
            neg_ &= ~(1u << k);
            return std::string(n ? "an_" : "am_");
        };
        for (const std::string& A : arrays_)
            if (mfma_array(A))
                for (int k : pairs(op)) {
                    const int k1 = k | (1 << op.pos);
                    xy.push_back({rk(A, k), rk(A, k1), col(k), col(k1)});
                }
        const int n = (int)xy.size();
        const int at = (int)(&op - p_->ops.data()) - aop0_, ab = ablock_of_[at];
        o_ << "    {\n      const float am_ = __uint_as_float(am" << agroup_of_[at] << "_ ^ as_);\n";
        if (neg) o_ << "      const float an_ = __uint_as_float(am" << agroup_of_[at] << "_ ^ ~as_ & 0x80000000u);\n";
        for (int i = 0; i < n; ++i)
            o_ << "      qsv_v4f c" << i << "_ = __builtin_amdgcn_mfma_f32_4x4x1f32(" << xy[i].a0 << ", " << xy[i].first
               << ".x, qsv_v4f{0.f, 0.f, 0.f, 0.f}, 4, " << ab << ", 0);\n";
        for (int st = 1; st < 4; ++st)
            for (int i = 0; i < n; ++i) {
                const std::string src = st == 1 ? xy[i].first + ".y" : st == 2 ? xy[i].second + ".x" : xy[i].second + ".y";
                o_ << "      c" << i << "_ = __builtin_amdgcn_mfma_f32_4x4x1f32(" << (st == 1 ? xy[i].a0 : xy[i].a1) << ", " << src << ", c" << i
                   << "_, 4, " << ab + st << ", 0);\n";
            }
        for (int i = 0; i < n; ++i)
            o_ << "      " << xy[i].first << " = make_float2(c" << i << "_[0], c" << i << "_[1]); " << xy[i].second
               << " = make_float2(c" << i << "_[2], c" << i << "_[3]);\n";
        o_ << "    }\n";
    }

    void emit_pair_op(const DOp& op, const std::string& A) {
        for (int k : pairs(op)) {
            const int k1 = k | (1 << op.pos);
            const std::string x = rk(A, k), y = rk(A, k1);
            o_ << "      { const f2 x = " << x << ", y = " << y << ";\n";
            switch (op.kind) {
            case OP_U2:
                o_ << "        " << x << " = make_float2(m0r * x.x - m0i * x.y + m1r * y.x - m1i * y.y, "
                   << "m0r * x.y + m0i * x.x + m1r * y.y + m1i * y.x);\n"
                   << "        " << y << " = make_float2(m2r * x.x - m2i * x.y + m3r * y.x - m3i * y.y, "
                   << "m2r * x.y + m2i * x.x + m3r * y.y + m3i * y.x); }\n";
                break;
            case OP_REAL:
                o_ << "        " << x << " = make_float2(m0r * x.x + m1r * y.x, m0r * x.y + m1r * y.y);\n"
                   << "        " << y << " = make_float2(m2r * x.x + m3r * y.x, m2r * x.y + m3r * y.y); }\n";
                break;
            case OP_RXL:
                o_ << "        " << x << " = make_float2(al * x.x - be * y.y, al * x.y + be * y.x);\n"
                   << "        " << y << " = make_float2(al * y.x - be * x.y, al * y.y + be * x.x); }\n";
                break;
            case OP_SWAP:
                o_ << "        " << x << " = y; " << y << " = x; }\n";
                break;
            }
        }
    }

    // The rotation of a core, in place: three shears of one multiply-add per
    // amplitude component each. The backward is bound by vector instructions;
    // with shears and one vector of phases for four qubits the longest pass of
    // the 20-qubit ladder has 18,500 of them instead of 25,700, and its backward
    // takes 5.4 ms instead of 6.8 (batch 64). Two multiply-adds by tan(phi) and a
    // late scale would do, but need a second form for |tan| > 1: as a branch between
    // two forms it cost about 30 register copies and 45 more VGPRs, as a conditional
    // swap before one form it saves 5% of the pass's instructions on average.
    void emit_shear(const DOp& op) {
        o_ << "    const float* M_ = " << mat_ptr(op.mat) << ";\n    const float a_ = M_[0], b_ = M_[1];\n";
        for (const std::string& A : arrays_)
            for (int step = 0; step < 3; ++step)
                for (int k : pairs(op)) {
                    const std::string x = rk(A, k), y = rk(A, k | (1 << op.pos));
                    const std::string to = step == 1 ? y : x, from = step == 1 ? x : y;
                    const char* c = step == 1 ? "b_" : "a_";
                    const char* sg = step == 1 ? "" : "-";
                    o_ << "    " << to << ".x = fmaf(" << sg << c << ", " << from << ".x, " << to << ".x); " << to
                       << ".y = fmaf(" << sg << c << ", " << from << ".y, " << to << ".y);\n";
                }
    }

    // Waiting diagonals of the register qubits, one complex value per register index;
    // OP_DVEC2 adds the product with what rounding took off the value.
    void emit_dvec(const DOp& op) {
        const bool res = op.kind == OP_DVEC2;
        o_ << "    const float* M_ = " << mat_ptr(op.mat) << ";\n";
        for (int k = 0; k < kRegs; ++k) {
            const int e = k & op.pos;
            if (!e) continue;
            o_ << "    { const float r_ = M_[" << 2 * e << "], i_ = M_[" << 2 * e + 1 << "];\n";
            if (res) o_ << "      const float u_ = M_[" << 32 + 2 * e << "], v_ = M_[" << 33 + 2 * e << "];\n";
            for (const std::string& A : arrays_) {
                o_ << "      { const f2 x = " << rk(A, k) << "; " << rk(A, k) << " = ";
                if (res)
                    o_ << "make_float2(fmaf(r_, x.x, fmaf(-i_, x.y, fmaf(u_, x.x, -v_ * x.y))), "
                          "fmaf(r_, x.y, fmaf(i_, x.x, fmaf(u_, x.y, v_ * x.x)))); }\n";
                else
                    o_ << "make_float2(r_ * x.x - i_ * x.y, r_ * x.y + i_ * x.x); }\n";
            }
            o_ << "    }\n";
        }
    }

    // Registers of a forward kernel that hold the negative of their amplitude:
    // a matrix instruction takes the sign along (negated A operand), everything
    // else has it applied first.
    uint32_t neg_ = 0;
    void apply_neg() {
        for (int k = 0; k < kRegs; ++k)
            if (neg_ >> k & 1)
                for (const std::string& A : arrays_)
                    o_ << "  " << rk(A, k) << " = make_float2(-" << rk(A, k) << ".x, -" << rk(A, k) << ".y);\n";
        neg_ = 0;
    }

    void emit_apply(const DOp& op) {
        if (op.kind != OP_SIGN && !use_mfma(op)) apply_neg();
        o_ << "  {\n";
        if (op.kind == OP_SHEAR) {
            emit_shear(op);
            o_ << "  }\n";
            return;
        }
        if (op.kind == OP_DVEC || op.kind == OP_DVEC2) {
            emit_dvec(op);
            o_ << "  }\n";
            return;
        }
        if (op.kind != OP_SIGN && op.kind != OP_SWAP) emit_matrix(op);
        if (op.kind == OP_SIGN) {
            // Uniform part folded at compile time. Per-thread part: one word per set
            // of terms that some register is in, the term's sign in its top bit, so a
            // flip is one instruction per component. (A word per register, from a mask
            // of all terms, took three.)
            std::vector<std::vector<int>> set_of(kRegs), sets;
            for (int k = 0; k < kRegs; ++k) {
                for (int i = 0; i < op.nterm; ++i)
                    if (p_->terms[op.term0 + i].mask >> k & 1) set_of[k].push_back(i);
                if (!set_of[k].empty() && std::find(sets.begin(), sets.end(), set_of[k]) == sets.end())
                    sets.push_back(set_of[k]);
            }
            for (int i = 0; i < op.nterm; ++i) {
                const DTerm& tm = p_->terms[op.term0 + i];
                o_ << "    const unsigned f" << i << "_ = ((unsigned)gT << " << 31 - tm.s0 << ")";
                for (int s : {tm.s1, tm.s2})
                    if (s >= 0) o_ << " & ((unsigned)gT << " << 31 - s << ")";
                o_ << ";\n";
            }
            for (size_t j = 0; j < sets.size(); ++j) {
                std::string w;
                for (int i : sets[j]) w += (w.empty() ? "f" : " ^ f") + I(i) + "_";
                o_ << "    const unsigned w" << j << "_ = " << w << ";\n";
            }
            const bool later = !bwd_ && (p_->opts.mfma & 1);  // matrix instructions take signs along
            if (later) neg_ ^= (uint32_t)op.pos & 0xFFFF;
            for (const std::string& A : arrays_)
                for (int k = 0; k < kRegs; ++k) {
                    const bool u = !later && (op.pos >> k & 1);
                    const std::string x = rk(A, k);
                    if (!set_of[k].empty()) {
                        const size_t j = std::find(sets.begin(), sets.end(), set_of[k]) - sets.begin();
                        o_ << "    " << x << " = qsv_flip(" << x << ", " << (u ? "~w" : "w") << j << "_);\n";
                    } else if (u) {
                        o_ << "    " << x << " = make_float2(-" << x << ".x, -" << x << ".y);\n";
                    }
                }
            o_ << "  }\n";
            return;
        }
        if (op.kind == OP_DIAG) {
            const std::string nc = nonreg_cond(op);
            if (!nc.empty()) o_ << "    if (" << nc << ") {\n";
            if (op.pos >= 0) {
                for (const std::string& A : arrays_)
                    for (int k = 0; k < kRegs; ++k) {
                        if (!reg_ok(op, k)) continue;
                        const bool hi = k >> op.pos & 1;
                        const std::string pr = hi ? "m3r" : "m0r", pi = hi ? "m3i" : "m0i";
                        o_ << "    { const f2 x = " << rk(A, k) << "; " << rk(A, k) << " = make_float2(" << pr
                           << " * x.x - " << pi << " * x.y, " << pr << " * x.y + " << pi << " * x.x); }\n";
                    }
            } else {
                o_ << "    const bool hb_ = (gT >> " << op.sh << ") & 1;\n"
                   << "    const float pr = hb_ ? m3r : m0r, pi = hb_ ? m3i : m0i;\n";
                for (const std::string& A : arrays_)
                    for (int k = 0; k < kRegs; ++k) {
                        if (!reg_ok(op, k)) continue;
                        o_ << "    { const f2 x = " << rk(A, k) << "; " << rk(A, k)
                           << " = make_float2(pr * x.x - pi * x.y, pr * x.y + pi * x.x); }\n";
                    }
            }
            if (!nc.empty()) o_ << "    }\n";
            o_ << "  }\n";
            return;
        }
        const std::string nc = nonreg_cond(op);
        if (op.kind == OP_SWAP && !nc.empty() && lane_ctl(op)) {
            // A swap under a per-lane control as selects: written as a branch,
            // the compiler keeps both orders of every pair live across the
            // divergent region (64 more VGPRs for psi and lambda).
            o_ << "    const bool c_ = " << nc << ";\n";
            for (const std::string& A : arrays_)
                for (int k : pairs(op)) {
                    const std::string x = rk(A, k), y = rk(A, k | (1 << op.pos));
                    o_ << "    { const f2 x = " << x << ", y = " << y << "; " << x << " = c_ ? y : x; " << y
                       << " = c_ ? x : y; }\n";
                }
            o_ << "  }\n";
            return;
        }
        if (!nc.empty()) o_ << "    if (" << nc << ") {\n";
        if (use_mfma(op)) emit_pairs_mfma(op);
        for (const std::string& A : arrays_)
            if (!use_mfma(op) || !mfma_array(A)) emit_pair_op(op, A);
        if (!nc.empty()) o_ << "    }\n";
        o_ << "  }\n";
    }

    void emit_grad(const DOp& op) {
        // two float32 accumulators (alternating terms), summed at the end
        const std::string gs = "g" + I(op.slot);
        const std::string g = "ga_";
        o_ << "  {\n    float ga_ = 0.f, gb_ = 0.f;\n";
        const std::string nc = nonreg_cond(op);
        if (op.kind == OP_GZ && op.pos < 0) {
            o_ << "    float h_ = 0.f;\n";
            if (!nc.empty()) o_ << "    if (" << nc << ") {\n";
            for (int k = 0; k < kRegs; ++k) {
                if (!reg_ok(op, k)) continue;
                o_ << "    h_ = fmaf(lm[" << k << "].x, ps[" << k << "].y, h_); h_ = fmaf(-lm[" << k
                   << "].y, ps[" << k << "].x, h_);\n";
            }
            if (!nc.empty()) o_ << "    }\n";
            o_ << "    " << gs << " = ((gT >> " << op.sh << ") & 1) ? -h_ : h_;\n  }\n";
            return;
        }
        if (!nc.empty()) o_ << "    if (" << nc << ") {\n";
        if (op.kind == OP_GZ) {
            for (int k = 0; k < kRegs; ++k) {
                if (!reg_ok(op, k)) continue;
                const std::string g = (k & 1) ? "gb_" : "ga_";
                const char* sg = (k >> op.pos & 1) ? "-" : "";
                o_ << "    " << g << " = fmaf(" << sg << "lm[" << k << "].x, ps[" << k << "].y, " << g << "); "
                   << g << " = fmaf(" << (sg[0] ? "" : "-") << "lm[" << k << "].y, ps[" << k << "].x, " << g
                   << ");\n";
            }
        } else {
            int alt = 0;
            for (int k : pairs(op)) {
                const std::string g = (alt++ & 1) ? "gb_" : "ga_";
                const int k1 = k | (1 << op.pos);
                const std::string l0 = rk("lm", k), l1 = rk("lm", k1), p0 = rk("ps", k), p1 = rk("ps", k1);
                if (op.kind == OP_GX)  // Im(conj(l0) p1) + Im(conj(l1) p0)
                    o_ << "    " << g << " = fmaf(" << l0 << ".x, " << p1 << ".y, " << g << "); " << g << " = fmaf(-"
                       << l0 << ".y, " << p1 << ".x, " << g << "); " << g << " = fmaf(" << l1 << ".x, " << p0
                       << ".y, " << g << "); " << g << " = fmaf(-" << l1 << ".y, " << p0 << ".x, " << g << ");\n";
                else  // GY: Re(conj(l1) p0) - Re(conj(l0) p1)
                    o_ << "    " << g << " = fmaf(" << l1 << ".x, " << p0 << ".x, " << g << "); " << g << " = fmaf("
                       << l1 << ".y, " << p0 << ".y, " << g << "); " << g << " = fmaf(-" << l0 << ".x, " << p1
                       << ".x, " << g << "); " << g << " = fmaf(-" << l0 << ".y, " << p1 << ".y, " << g << ");\n";
            }
        }
        if (!nc.empty()) o_ << "    }\n";
        o_ << "    " << gs << " = ga_ + gb_;\n  }\n";
    }

    // Gradient ops [a, b), taken at one point of the schedule.
    void emit_grads(int a, int b) {
        // Z components on several register qubits share their 16 products
        std::vector<int> zs;
        for (int i = a; i < b; ++i) {
            const DOp& op = p_->ops[i];
            if (op.kind == OP_GZ && op.pos >= 0 && op.ctl < 0) zs.push_back(i);
        }
        if (zs.size() >= 2) emit_joint_z(zs);
        else zs.clear();
        for (int i = a; i < b; ++i)
            if (std::find(zs.begin(), zs.end(), i) == zs.end()) emit_grad(p_->ops[i]);
        // Partials are reduced to one float32 per 16-lane row right away; rows are
        // combined in float64 at the end of the pass. Every lane that holds a sum
        // stores it (same value, same address): no branch, which keeps the
        // compiler's register allocation across the kernel intact.
        for (int i = a; i < b;) {
            const int sl = p_->ops[i].slot;
            bool four = i + 4 <= b;
            for (int j = 1; four && j < 4; ++j) four = p_->ops[i + j].slot == sl + j;
            if (four) {
                o_ << "  red4_[" << sl << "] = qsv_row_sum4(g" << sl << ", g" << sl + 1 << ", g" << sl + 2 << ", g" << sl + 3
                   << ");\n";
                i += 4;
            } else {
                o_ << "  red1_[" << sl << "] = qsv_row_sum(g" << sl << ");\n";
                ++i;
            }
        }
    }

    // Im<l|Z_q|psi> of the ops `zs` on different register qubits: the 16 products
    // Im(conj(l) psi) once, then sums over the other qubits and, qubit by qubit,
    // the difference of the halves and their sum (72 operations for four qubits
    // instead of 128).
    void emit_joint_z(const std::vector<int>& zs) {
        o_ << "  {\n";
        for (int k = 0; k < kRegs; ++k)
            o_ << "    const float z" << k << "_ = fmaf(lm[" << k << "].x, ps[" << k << "].y, -(lm[" << k << "].y * ps[" << k
               << "].x));\n";
        std::vector<std::string> v;
        for (int k = 0; k < kRegs; ++k) v.push_back("z" + I(k) + "_");
        std::vector<int> pos = {0, 1, 2, 3};  // register position of each index bit of v
        int id = 0;
        auto fold = [&](int i) {  // halves of v along index bit i: sums, and the sum of differences
            std::vector<std::string> sum;
            std::string d;
            for (int k = 0; k < (int)v.size(); ++k) {
                if (k >> i & 1) continue;
                const std::string &x = v[k], &y = v[k | (1 << i)];
                const std::string name = "y" + I(id++) + "_";
                o_ << "    const float " << name << " = " << x << " + " << y << ";\n";
                sum.push_back(name);
                d += (d.empty() ? "(" : " + (") + x + " - " + y + ")";
            }
            v = sum;
            pos.erase(pos.begin() + i);
            return d;
        };
        auto slots_on = [&](int p) {  // several where diagonal gates on one qubit lie between controlled ones
            std::vector<int> sl;
            for (int i : zs)
                if (p_->ops[i].pos == p) sl.push_back(p_->ops[i].slot);
            return sl;
        };
        for (int i = 0; i < (int)pos.size();) {
            if (slots_on(pos[i]).empty()) fold(i);
            else ++i;
        }
        while (!pos.empty()) {
            const std::vector<int> sl = slots_on(pos[0]);
            const std::string d = fold(0);
            o_ << "    g" << sl[0] << " = " << d << ";\n";
            for (size_t i = 1; i < sl.size(); ++i) o_ << "    g" << sl[i] << " = g" << sl[0] << ";\n";
        }
        o_ << "  }\n";
    }

    // Readout of the last forward pass (when epart is given): per tile and
    // qubit i, sum |a|^2 (1 - 2 bit_i) into epart[(b ntiles + tile) W + i].
    // Reduced values: the thread's total T, its sums S_r over registers with
    // register bit r set, and T on threads with thread-index bit j set; the
    // out-of-tile qubits take the tile total with the tile's sign.
    void emit_readout(const Layout& L) {
        const int nreg = kRegBits, ntb = (int)L.nonreg.size();
        const int nv = 1 + nreg + ntb, nw = threads_ / 64;
        o_ << "  if (epart) {\n    __shared__ double ered_[" << nw * nv << "];\n";
        o_ << "    float T_ = 0.f, S_[" << nreg << "] = {0.f, 0.f, 0.f, 0.f};\n";
        o_ << "    if (" << (guard_ ? "act" : "true") << ") {\n";
        for (int k = 0; k < kRegs; ++k) {
            o_ << "      { const float p_ = a[" << k << "].x * a[" << k << "].x + a[" << k << "].y * a[" << k
               << "].y; T_ += p_;";
            for (int r = 0; r < nreg; ++r)
                if (k >> r & 1) o_ << " S_[" << r << "] += p_;";
            o_ << " }\n";
        }
        o_ << "    }\n";
        o_ << "    double v_[" << nv << "];\n    v_[0] = T_;\n";
        for (int r = 0; r < nreg; ++r) o_ << "    v_[" << 1 + r << "] = S_[" << r << "];\n";
        for (int j = 0; j < ntb; ++j)
            o_ << "    v_[" << 1 + nreg + j << "] = ((t >> " << j << ") & 1) ? (double)T_ : 0.0;\n";
        o_ << "    for (int k = 0; k < " << nv << "; ++k) { const double r_ = qsv_wave_sum(v_[k]); "
           << "if (lane == 0) ered_[wave * " << nv << " + k] = r_; }\n";
        o_ << "    __syncthreads();\n";
        o_ << "    const int* eq_ = " << name_ << "_eq;\n";
        o_ << "    for (int i = t; i < " << W_ << "; i += " << threads_ << ") {\n"
           << "      double tot = 0.0, part_ = 0.0;\n"
           << "      for (int w = 0; w < " << nw << "; ++w) { tot += ered_[w * " << nv << "]; "
           << "if (eq_[2 * i] != 2) part_ += ered_[w * " << nv << " + eq_[2 * i + 1]]; }\n"
           << "      const double e = eq_[2 * i] == 2 ? (((base >> eq_[2 * i + 1]) & 1) ? -tot : tot)"
           << " : tot - 2.0 * part_;\n"
           << "      epart[((size_t)b * " << (1u << (W_ - m_)) << "u + tis) * " << W_ << " + i] = e;\n    }\n  }\n";
    }

    // per qubit of the readout: kind (0 register bit, 1 thread bit, 2 out-of-tile)
    // and the reduced value's index (kinds 0, 1) or the index-bit shift (kind 2)
    std::string readout_table(const Layout& L) const {
        std::ostringstream e;
        e << "__device__ const int " << name_ << "_eq[" << 2 * W_ << "] = {";
        for (int i = 0; i < W_; ++i) {
            const int sh = W_ - 1 - i;
            int kind = 2, idx = sh;
            for (int r = 0; r < kRegBits; ++r)
                if (lq(L.reg[r]) == sh) { kind = 0; idx = 1 + r; }
            for (int j = 0; j < (int)L.nonreg.size(); ++j)
                if (lq(L.nonreg[j]) == sh) { kind = 1; idx = 1 + kRegBits + j; }
            e << (i ? "," : "") << kind << "," << idx;
        }
        e << "};\n";
        return e.str();
    }

    void emit_kernel(const std::string& name) {
        name_ = name;
        const int tb = W_ - m_;
        if (last_fwd_) {
            o_ << readout_table(nat_layout());
        }
        if (bwd_ && ps_->n_gout) {
            // gradient outputs of this pass: ordinal, axis, component slots x/y/z, matrix slot
            o_ << "__device__ const int " << name << "_out[" << 6 * ps_->n_gout << "] = {";
            for (int j = 0; j < ps_->n_gout; ++j) {
                const DGOut& go = p_->gouts[ps_->gout0 + j];
                o_ << (j ? "," : "") << go.ord << "," << go.axis << "," << go.c0 << "," << go.c1 << ","
                   << go.c2 << "," << go.mat;
            }
            o_ << "};\n";
        }
        o_ << "extern \"C\" __global__ void __launch_bounds__(" << threads_ << ") " << name << "(";
        if (bwd_)
            o_ << "const f2* __restrict__ psiN, f2* __restrict__ psi, f2* __restrict__ lam, "
                  "const double* __restrict__ gout, const float* __restrict__ mats, int n_shared, int n_ps, "
                  "double* __restrict__ part, int B)\n{\n";
        else
            o_ << "f2* __restrict__ state, const float* __restrict__ mats, int n_shared, int n_ps"
               << (last_fwd_ ? ", double* __restrict__ epart" : "") << ")\n{\n";
        o_ << "  __shared__ f2 lds[" << (1 << m_) << "];\n";
        int ng = bwd_ ? ps_->n_gslots : 0;
        const int nw = threads_ / 64;
        // per-row float32 partials of every gradient slot: [wave * 4 + row][slot]
        if (bwd_ && ng) o_ << "  __shared__ float red[" << nw * 4 * ng << "];\n";
        o_ << "  const int t = threadIdx.x;\n";
        if (guard_) o_ << "  const bool act = t < " << T_ << ";\n";
        // Workgroups are dealt to the chip's 8 XCDs in turn (workgroup i to XCD
        // i mod 8), each with its own L2. When the tile count divides by 8, XCD x
        // takes the contiguous tile range [x n/8, (x+1) n/8): the tiles one XCD
        // holds at a time are then neighbours in the state (adjacent runs of the
        // lowest out-of-tile bits), not tiles 8 apart. 28 qubits: 54.2 -> 51.7 ms
        // per step; neutral on the ALU-bound passes.
        o_ << "  const unsigned tile = (gridDim.x & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (gridDim.x >> 3) + "
              "(blockIdx.x >> 3);\n"
           << "  const int b = (int)(tile >> " << tb << ");\n"
           << "  const int tis = (int)(tile & " << hex((1u << tb) - 1) << ");\n";
        {
            std::vector<int> pos;
            for (int k = 0; k < tb; ++k) pos.push_back(ps_->oq[k]);
            o_ << "  const int base = " << (tb ? scatter("tis", pos) : "0") << ";\n";
        }
        o_ << "  const size_t off = (size_t)b << " << W_ << ";\n"
           << "  const float* mp = mats + ((size_t)n_shared + (size_t)b * n_ps) * 8;\n"
           << "  (void)mp;\n";
        plan_a_operands();
        const Layout nat = nat_layout();
        lds_own_ = false;
        // With tile bit 0 = amplitude bit 0 in registers 0 and 1 of each pair,
        // a thread moves its amplitudes as 16-byte pairs when the array is
        // 16-byte aligned (a wave-uniform test; 8-byte aligned arrays take
        // single-amplitude accesses).
        const bool v16 = lq(0) == 0;
        Layout cur = nat;
        o_ << "  int gT = " << gT_expr(cur) << ";\n";
        for (const std::string& A : arrays_) o_ << "  f2 " << A << "[16];\n";
        if (guard_)
            for (const std::string& A : arrays_)
                o_ << "  for (int k = 0; k < 16; ++k) " << A << "[k] = make_float2(0.f, 0.f);\n";
        // Buffer accesses where a sample's bytes fit 32 bits: a byte offset from
        // the thread index, shared by all accesses and by psi and lambda, plus a
        // scalar constant per access, no address arithmetic (pointers take two
        // 64-bit additions' worth of vector instructions each).
        const bool buf = W_ <= kMaxBufferQubits;
        auto open = [&](const std::string& name, const std::string& ptr) {
            return buf ? "const __amdgpu_buffer_rsrc_t " + name + "b_ = qsv_buf(" + ptr + ", " + I(8LL << W_) + "u); " : std::string();
        };
        // Non-temporal where the arrays a launch passes over exceed the 256 MB Infinity
        // Cache twice: nothing of them is left when the next pass comes (28-qubit ring,
        // 2.1 GB a state: 47.4 -> 45.4 ms per step; 4-layer rings' backward, 0.5 GB of psi
        // and lambda: 2.36 -> 2.31 ms, 1.1 GB: 4.24 -> 4.07). Below, passes find part of
        // them there (16-qubit ring, batch 256, 0.13 GB a state: 1.93 -> 2.08 ms with
        // them; 21 qubits, batch 7, forward: 760 -> 857 us).
        const bool nt = buf && v16;
        if (nt)
            o_ << "  const bool nt_ = gridDim.x >= " << stream_tiles(m_, (int)arrays_.size()) << "u;\n";
        // by alignment (8 bytes: s1, 16: s2) and size (s3)
        auto by_access = [&](const std::string& ptr, const std::string& s1, const std::string& s2, const std::string& s3) {
            const std::string two = "if (((qsv_uptr)(" + ptr + ") & 15) != 0) { " + s1 + "} else ";
            return two + (nt ? "if (nt_) { " + s3 + "} else { " + s2 + "}" : "{ " + s2 + "}");
        };
        auto gload = [&](const std::string& A, const std::string& src) {
            std::string s1, s2, s3;
            for (int k = 0; k < kRegs; ++k) {
                s1 += A + "[" + I(k) + "] = ";
                if (buf) s1 += "qsv_ld2(" + A + "b_, gT << 3, " + I(gR(cur, k) * 8) + "); ";
                else s1 += src + "[gT + " + I(gR(cur, k)) + "]; ";
            }
            if (!v16) return "{ " + open(A, src) + s1 + "}";
            for (int k = 0; k < kRegs; k += 2) {
                auto pair = [&](const std::string& load) {
                    return "{ const float4 v_ = " + load + "; " + A + "[" + I(k) + "] = make_float2(v_.x, v_.y); " + A + "[" +
                           I(k + 1) + "] = make_float2(v_.z, v_.w); } ";
                };
                const std::string at = "(" + A + "b_, gT << 3, " + I(gR(cur, k) * 8) + ")";
                s2 += pair(buf ? "qsv_ld4<0>" + at
                               : "*reinterpret_cast<const float4*>(" + src + " + gT + " + I(gR(cur, k)) + ")");
                if (nt) s3 += pair("qsv_ld4<1>" + at);
            }
            return "{ " + open(A, src) + by_access(src, s1, s2, s3) + " }";
        };
        auto gstore = [&](const std::string& A, const std::string& dst) {
            std::string s1, s2, s3;
            for (int k = 0; k < kRegs; ++k) {
                const std::string v = A + "[" + I(k) + "]";
                if (buf) s1 += "qsv_st2(" + v + ", " + A + "b_, gT << 3, " + I(gR(cur, k) * 8) + "); ";
                else s1 += dst + "[gT + " + I(gR(cur, k)) + "] = " + v + "; ";
            }
            if (!v16) return "{ " + open(A, dst) + s1 + "}";
            for (int k = 0; k < kRegs; k += 2) {
                const std::string x = A + "[" + I(k) + "]", y = A + "[" + I(k + 1) + "]";
                const std::string v = "make_float4(" + x + ".x, " + x + ".y, " + y + ".x, " + y + ".y)";
                const std::string at = "(" + v + ", " + A + "b_, gT << 3, " + I(gR(cur, k) * 8) + "); ";
                if (buf) s2 += "qsv_st4<0>" + at;
                else s2 += "*reinterpret_cast<float4*>(" + dst + " + gT + " + I(gR(cur, k)) + ") = " + v + "; ";
                if (nt) s3 += "qsv_st4<1>" + at;
            }
            return "{ " + open(A, dst) + by_access(dst, s1, s2, s3) + " }";
        };
        const int flags = ps_->flags;
        if (!bwd_ && (flags & PF_INIT_FWD)) {
            // The first pass generates the product state of the leading 1-qubit
            // gates instead of loading it: amplitude idx is the product over
            // qubits q of column 0 of q's prefix matrix, entry bit_q(idx).
            o_ << "  f2* st = state + off;\n  {\n    f2 P_ = make_float2(1.f, 0.f);\n";
            auto vq = [&](int q) {
                const int slot = p_->prefix_mat[q];
                return slot >= 0 ? "mats + " + I(8LL * slot) : "mp + " + I(8LL * (-slot - 1));
            };
            std::vector<int> reg_shift(kRegBits);
            for (int r = 0; r < kRegBits; ++r) reg_shift[r] = lq(cur.reg[r]);
            for (int q = 0; q < W_; ++q) {
                const int sh = W_ - 1 - q;
                if (std::find(reg_shift.begin(), reg_shift.end(), sh) != reg_shift.end()) continue;
                o_ << "    { const float* v_ = " << vq(q) << "; const int bt_ = (gT >> " << sh << ") & 1;\n"
                   << "      const f2 u_ = bt_ ? make_float2(v_[4], v_[5]) : make_float2(v_[0], v_[1]);\n"
                   << "      P_ = make_float2(P_.x * u_.x - P_.y * u_.y, P_.x * u_.y + P_.y * u_.x); }\n";
            }
            // register qubits: a[k] = P_ * prod_r v_r[bit r of k], built as a doubling tree
            o_ << "    a[0] = P_;\n";
            for (int r = 0; r < kRegBits; ++r) {
                const int q = W_ - 1 - reg_shift[r];
                o_ << "    { const float* v_ = " << vq(q) << ";\n"
                   << "      const f2 u0_ = make_float2(v_[0], v_[1]), u1_ = make_float2(v_[4], v_[5]);\n";
                for (int k = (1 << r) - 1; k >= 0; --k) {
                    const int k1 = k | (1 << r);
                    o_ << "      a[" << k1 << "] = make_float2(a[" << k << "].x * u1_.x - a[" << k << "].y * u1_.y, a["
                       << k << "].x * u1_.y + a[" << k << "].y * u1_.x);\n"
                       << "      a[" << k << "] = make_float2(a[" << k << "].x * u0_.x - a[" << k << "].y * u0_.y, a["
                       << k << "].x * u0_.y + a[" << k << "].y * u0_.x);\n";
                }
                o_ << "    }\n";
            }
            o_ << "  }\n";
        } else if (!bwd_) {
            o_ << "  f2* st = state + off;\n  " << act(gload("a", "st")) << "\n";
        } else if (flags & PF_FIRST_BWD) {
            o_ << "  " << act(gload("ps", "(psiN + off)")) << "\n";
            // lambda = D psi with D(idx) = G0 - 2 sum_{i: bit_i(idx) = 1} g_i
            o_ << "  {\n    const double* g_ = gout + (size_t)b * " << W_ << ";\n"
               << "    double G0 = 0.0, DT = 0.0;\n"
               << "    for (int i = 0; i < " << W_ << "; ++i) { const double gi = g_[i]; G0 += gi; "
               << "if ((gT >> (" << W_ - 1 << " - i)) & 1) DT += gi; }\n";
            for (int p = 0; p < kRegBits; ++p)
                o_ << "    const double gp" << p << " = g_[" << W_ - 1 - lq(cur.reg[p]) << "];\n";
            for (int k = 0; k < kRegs; ++k) {
                std::string dr = "DT";
                for (int p = 0; p < kRegBits; ++p)
                    if (k >> p & 1) dr += " + gp" + I(p);
                o_ << "    { const float d = (float)(G0 - 2.0 * (" << dr << ")); lm[" << k << "] = make_float2(d * ps["
                   << k << "].x, d * ps[" << k << "].y); }\n";
            }
            o_ << "  }\n";
        } else {
            o_ << "  " << act(gload("ps", "(psi + off)") + gload("lm", "(lam + off)")) << "\n";
        }
        if (bwd_ && ng) {
            for (int j = 0; j < ng; ++j) o_ << "  float g" << j << " = 0.f;\n";
        }
        o_ << "  const int wave = t >> 6, lane = t & 63; (void)wave; (void)lane;\n";
        const bool write_back = !bwd_ || !(flags & PF_LAST_BWD);
        const std::vector<Layout> lays = choose_waves(nat, write_back);
        if (bwd_ && ng) {
            // this lane's row of partials, and the same with the lane's bank added
            o_ << "  float* const red1_ = red + (wave * 4 + (lane >> 4)) * " << ng << ";\n"
               << "  float* const red4_ = red1_ + ((lane >> 2) & 3); (void)red4_;\n";
        }
        for (int s = 0; s < ps_->n_stages; ++s) {
            const DStage& st = p_->stages[ps_->stage0 + s];
            const Layout& L = lays[s];
            if (!same(L, cur)) {
                apply_neg();
                emit_exchange(cur, L);
                cur = L;
            }
            lay_ = &cur;
            for (int oi = st.op0; oi < st.op1;) {
                int oe = oi;
                while (oe < st.op1 && is_grad_op(p_->ops[oe].kind)) ++oe;
                if (oe == oi) {
                    need_a_group(oi);
                    emit_apply(p_->ops[oi++]);
                }
                else emit_grads(oi, oe);
                oi = std::max(oi, oe);
            }
        }
        lay_ = nullptr;  // cur goes out of scope with this kernel
        apply_neg();
        if (write_back) {
            if (!same(cur, nat)) {
                emit_exchange(cur, nat);
                cur = nat;
            }
            o_ << "  " << act(bwd_ ? gstore("ps", "(psi + off)") + gstore("lm", "(lam + off)") : gstore("a", "st"))
               << "\n";
        }
        if (last_fwd_) emit_readout(cur);
        if (bwd_ && ng) {
            o_ << "  __syncthreads();\n";
            o_ << "  {\n    __shared__ double cs_[" << ng << "];\n";
            o_ << "    for (int j = t; j < " << ng << "; j += " << threads_ << ") {\n"
               << "      double s = 0.0;\n";
            for (int r = 0; r < nw * 4; ++r) o_ << "      s += (double)red[" << r * ng << " + j];\n";
            o_ << "      cs_[j] = s;\n    }\n    __syncthreads();\n";
            o_ << "    const int* out_ = " << name << "_out;\n"
               << "    for (int j = t; j < " << ps_->n_gout << "; j += " << threads_ << ") {\n"
               << "      const int* e = out_ + 6 * j;\n"
               << "      double v;\n"
               << "      if (e[1] < 0) v = cs_[e[2]];\n"
               << "      else v = qsv_chain_grad(e[5] >= 0 ? mats + 8 * (size_t)e[5] : mp + 8 * (size_t)(-e[5] - 1), "
                  "e[1], e[2] >= 0 ? cs_[e[2]] : 0.0, e[3] >= 0 ? cs_[e[3]] : 0.0, e[4] >= 0 ? cs_[e[4]] : 0.0);\n"
               << "      part[((size_t)e[0] * B + b) * " << (1u << tb) << "u + tis] = v;\n    }\n  }\n";
        }
        o_ << "}\n\n";
    }
};

std::string arch_of_device() {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return "";
    return prop.gcnArchName;
}

uint64_t fnv1a(const std::string& s) {
    uint64_t h = 1469598103934665603ull;
    for (unsigned char c : s) { h ^= c; h *= 1099511628211ull; }
    return h;
}

const char* const kOpts[] = {"-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};

std::string cache_path(const std::string& src, const std::string& arch) {
    const char* dir = std::getenv("QSV_JIT_CACHE");
    if (!dir || !*dir) return "";
    char b[40];
    // the tag changes whenever the compiler options below change
    std::snprintf(b, sizeof b, "%016llx", (unsigned long long)fnv1a(src + "|" + arch + "|opts2"));
    return std::string(dir) + "/qsv_" + b + ".co";
}

bool read_file(const std::string& path, std::vector<char>& out) {
    std::ifstream f(path, std::ios::binary);
    if (!f) return false;
    out.assign(std::istreambuf_iterator<char>(f), std::istreambuf_iterator<char>());
    return !out.empty();
}

void write_cache(const std::string& path, const std::vector<char>& code) {
    if (path.empty()) return;
    const std::string tmp = path + ".tmp" + std::to_string((long long)getpid()) + "_" +
                            std::to_string((long long)std::hash<std::thread::id>()(std::this_thread::get_id()));
    std::ofstream f(tmp, std::ios::binary);
    f.write(code.data(), (std::streamsize)code.size());
    f.close();
    std::rename(tmp.c_str(), path.c_str());
}

// The ROCm clang driver, if installed (QSV_JIT_CLANG overrides; "none" disables).
std::string find_clang() {
    const char* env = std::getenv("QSV_JIT_CLANG");
    if (env && *env) return std::string(env) == "none" ? "" : env;
    const char* rp = std::getenv("ROCM_PATH");
    const std::string cands[] = {std::string(rp ? rp : "/opt/rocm") + "/llvm/bin/clang++",
                                 "/opt/rocm/llvm/bin/clang++"};
    for (const auto& c : cands)
        if (access(c.c_str(), X_OK) == 0) return c;
    return "";
}

extern "C" char** environ;

// Compile sources in parallel child processes of the clang driver.
int compile_children(const std::string& clang, const std::vector<std::string>& srcs,
                     const std::string& arch, std::vector<std::vector<char>>& codes,
                     std::vector<int>& todo, std::string& err) {
    const char* tmpenv = std::getenv("TMPDIR");
    std::string tmpl = std::string(tmpenv && *tmpenv ? tmpenv : "/tmp") + "/qsv_jit_XXXXXX";
    std::vector<char> dirbuf(tmpl.begin(), tmpl.end());
    dirbuf.push_back(0);
    if (!mkdtemp(dirbuf.data())) {
        err = "mkdtemp failed";
        return QSV_ERR_HIP;
    }
    const std::string dir = dirbuf.data();
    const int maxpar = std::max(1, std::min<int>(16, (int)std::thread::hardware_concurrency()));
    const std::string arch_opt = "--offload-arch=" + arch;
    int rc = QSV_OK;
    size_t next = 0;
    std::vector<std::pair<pid_t, int>> running;
    auto paths = [&](int i, const char* ext) { return dir + "/k" + std::to_string(i) + ext; };
    while ((next < todo.size() || !running.empty()) && rc == QSV_OK) {
        while (next < todo.size() && (int)running.size() < maxpar) {
            const int i = todo[next++];
            {
                std::ofstream f(paths(i, ".hip"));
                f << srcs[i];
            }
            const std::string in = paths(i, ".hip"), out = paths(i, ".co"), log = paths(i, ".log");
            std::vector<std::string> args = {clang, "-x", "hip", arch_opt, "--cuda-device-only",
                                             "--no-gpu-bundle-output", "-O3", "-std=c++17",
                                             "-include", "hip/hip_runtime.h",
                                             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                                             "-mllvm", "-amdgpu-mfma-vgpr-form=1", "-o", out, in};
            std::vector<char*> argv;
            for (auto& a : args) argv.push_back(&a[0]);
            argv.push_back(nullptr);
            posix_spawn_file_actions_t fa;
            posix_spawn_file_actions_init(&fa);
            posix_spawn_file_actions_addopen(&fa, 1, log.c_str(), O_WRONLY | O_CREAT | O_TRUNC, 0644);
            posix_spawn_file_actions_adddup2(&fa, 1, 2);
            pid_t pid;
            const int e = posix_spawn(&pid, clang.c_str(), &fa, nullptr, argv.data(), environ);
            posix_spawn_file_actions_destroy(&fa);
            if (e != 0) {
                err = "cannot start " + clang;
                rc = QSV_ERR_HIP;
                break;
            }
            running.emplace_back(pid, i);
        }
        if (running.empty()) break;
        int status = 0;
        const pid_t done = waitpid(-1, &status, 0);
        if (done < 0) {
            err = "waitpid failed";
            rc = QSV_ERR_HIP;
            break;
        }
        for (size_t r = 0; r < running.size(); ++r) {
            if (running[r].first != done) continue;
            const int i = running[r].second;
            running.erase(running.begin() + (long)r);
            if (!WIFEXITED(status) || WEXITSTATUS(status) != 0 || !read_file(paths(i, ".co"), codes[i])) {
                std::vector<char> log;
                read_file(paths(i, ".log"), log);
                err = "kernel compile failed: " + std::string(log.begin(), log.end()).substr(0, 2000);
                rc = QSV_ERR_HIP;
            }
            break;
        }
    }
    for (auto& r : running) waitpid(r.first, nullptr, 0);
    for (size_t i = 0; i < srcs.size(); ++i)
        for (const char* ext : {".hip", ".co", ".log"}) std::remove(paths((int)i, ext).c_str());
    rmdir(dir.c_str());
    return rc;
}

}  // namespace

// Compile one group of kernels (source) for `arch` with hipRTC.
static int compile_group(const std::string& src, const std::string& arch, std::vector<char>& code,
                         std::string& log) {
    hiprtcProgram prog;
    if (hiprtcCreateProgram(&prog, src.c_str(), "qsv_jit.hip", 0, nullptr, nullptr) != HIPRTC_SUCCESS) {
        log = "hiprtcCreateProgram failed";
        return QSV_ERR_HIP;
    }
    std::vector<const char*> opts(std::begin(kOpts), std::end(kOpts));
    const std::string arch_opt = "--offload-arch=" + arch;
    opts.push_back(arch_opt.c_str());
    const hiprtcResult r = hiprtcCompileProgram(prog, (int)opts.size(), opts.data());
    size_t n = 0;
    hiprtcGetProgramLogSize(prog, &n);
    if (n > 1) {
        log.resize(n);
        hiprtcGetProgramLog(prog, &log[0]);
    }
    if (r != HIPRTC_SUCCESS) {
        hiprtcDestroyProgram(&prog);
        return QSV_ERR_HIP;
    }
    hiprtcGetCodeSize(prog, &n);
    code.resize(n);
    hiprtcGetCode(prog, code.data());
    hiprtcDestroyProgram(&prog);
    return QSV_OK;
}

std::string jit_source(const qsv_plan_t* p, std::vector<JitKernelRef>& refs, int max_ops_per_group) {
    Gen g(p);
    std::string all;
    refs.clear();
    int group = 0, ops_in_group = 0;
    for (int which = 0; which < 2; ++which) {
        const auto& passes = which == 0 ? p->fwd_pass : p->bwd_pass;
        for (int i = 0; i < (int)passes.size(); ++i) {
            int nops = 0;
            for (int s = passes[i].stage0; s < passes[i].stage0 + passes[i].n_stages; ++s)
                nops += p->stages[s].op1 - p->stages[s].op0;
            if (ops_in_group && ops_in_group + nops > max_ops_per_group) {
                ++group;
                ops_in_group = 0;
            }
            ops_in_group += nops;
            JitKernelRef r;
            r.which = which;
            r.pass = i;
            r.group = group;
            r.source = g.kernel(which, i, r.name);
            refs.push_back(r);
        }
    }
    for (auto& r : refs) all += r.source;
    return g.prelude() + all;
}

int jit_compile(const qsv_plan_t* p, const std::string& arch_in, JitModules& out, std::string& err) {
    std::vector<JitKernelRef> refs;
    Gen g(p);
    jit_source(p, refs, 1);  // one kernel per compilation unit: compiled in parallel
    const std::string arch = arch_in.empty() ? arch_of_device() : arch_in;
    if (arch.empty()) {
        err = "cannot determine the device architecture";
        return QSV_ERR_HIP;
    }
    int ngroups = refs.empty() ? 0 : refs.back().group + 1;
    std::vector<std::string> srcs(ngroups, g.prelude());
    for (auto& r : refs) srcs[r.group] += r.source;
    std::vector<std::vector<char>> codes(ngroups);
    std::vector<int> todo;
    for (int i = 0; i < ngroups; ++i)
        if (!read_file(cache_path(srcs[i], arch), codes[i])) todo.push_back(i);
    const std::string clang = find_clang();
    if (!todo.empty() && !clang.empty()) {
        int rc = compile_children(clang, srcs, arch, codes, todo, err);
        if (rc != QSV_OK) return rc;
    } else {
        for (int i : todo) {
            std::string log;
            if (compile_group(srcs[i], arch, codes[i], log) != QSV_OK) {
                err = "hipRTC compile failed: " + log.substr(0, 2000);
                return QSV_ERR_HIP;
            }
        }
    }
    for (int i : todo) write_cache(cache_path(srcs[i], arch), codes[i]);
    out.codes = std::move(codes);
    out.refs = std::move(refs);
    out.arch = arch;
    return QSV_OK;
}

}  // namespace qsv
