// Operation lists of a plan in the form that the direct interpreter of the pass kernel reads.
#pragma once
#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "qsv_gate_asm.h"
#include "qsv_plan.h"

namespace qsv {

struct DirectOp {
    uint32_t code;   // byte offset of the operation's code in its interpreter
    uint32_t arg;    // unitaries: index in execution order; conditions: mask of index bits; lane exchange: mask of the
                     // lane number; transposes: offset / 64 of the target layout's code | flags << 16
};
static_assert(sizeof(DirectOp) == sizeof(Op), "both forms take the same room");

struct DirectPass {
    int begin;           // first operation
    int s_in, s_out;     // register layouts of the load and the store
    int first_mat;       // table entry of the first unitary (0 if none)
    int first_u;         // its index (0 if none)
    int n_ops, n_mats;   // operations and table entries of the pass
};

struct DirectPlan {
    std::vector<DirectOp> ops;   // never more than the plan has, but for the scalars of groups and the sums of pairs
    std::vector<DirectPass> passes;
};

// What the paired interpreter does around a unitary (see sum_handlers in the generator): the axes, 0..2 for X, Y, Z, of
// the circuit's rotation slots; none: no sums.
struct SumAxes {
    int count = 0, axis[4] = {};
};

inline SumAxes sum_axes(const qsv_circuit& c) {
    SumAxes a;
    if (c.reupload) a.axis[a.count++] = QSV_RX - 1;
    for (int r = 0; r < c.n_rot; ++r) a.axis[a.count++] = c.rot[r] - 1;
    return a;
}

// Lowers one operation list (a pass: OP_LOAD ... OP_END) onto out; false if it holds something the direct
// interpreter has no code for (never planned for tiles of one row).  rows: what gradient rows may do to a unitary.
// sums (the paired interpreter): the sums to be taken.  groups: Plan::groups, NULL or empty: the scalars are in the matrices.
enum class Rows { none, replace, turn };   // replace its matrix, or multiply by another before it

template <class Code>
bool lower_pass_as(const Op* ops, int count, Rows rows, const SumAxes& sums, const std::vector<int32_t>* groups,
                   DirectPlan* out) {
    constexpr bool pair = std::is_same<Code, paired>::value;
    const bool scaled = groups && !groups->empty();
    // the group of unitary k: the last start that is not behind it
    auto group_of = [&](int k) { return (int)(std::upper_bound(groups->begin(), groups->end(), k) - groups->begin()) - 1; };
    DirectPass dp;
    dp.begin = (int)out->ops.size();
    dp.s_in = dp.s_out = -1;
    dp.first_mat = dp.first_u = -1;
    dp.n_mats = 0;
    int s = -1;
    uint32_t rungs = 0;          // CZ rungs inside the run, collected: neighbouring ones go in one operation
    auto put = [&](uint32_t code, uint32_t arg) { out->ops.push_back({code, arg}); };
    auto flush = [&]() {
        if (rungs) put(Code::kCz[rungs], 0);
        rungs = 0;
    };
    for (int k = 0; k < count; ++k) {
        const Op& o = ops[k];
        if (o.kind == OP_CZ_REG) {
            if (o.a > 2 || o.b != o.a + 1) return false;
            rungs ^= 1u << o.a;
            continue;
        }
        // the CZ gates commute with each other, so rungs may wait for the next gate that is none
        if (o.kind != OP_CZ_MIX && o.kind != OP_CZ_LANE) flush();
        switch (o.kind) {
            case OP_LOAD:
                if (k != 0) return false;
                dp.s_in = s = o.a;
                break;
            case OP_U:
                if (o.a > 3) return false;
                if (dp.first_u < 0) {
                    dp.first_u = o.arg;
                    dp.first_mat = o.arg + (scaled ? group_of(o.arg) : 0);
                }
                ++dp.n_mats;
                if (scaled ? o.c || rows == Rows::replace : rows == Rows::turn) return false;
                if constexpr (pair) {
                    if (sums.count < 1 || o.c) return false;
                    if (sums.count == 2) put(Code::kBefore[o.a][sums.axis[1]], 0);
                    put(Code::kU[o.a], (uint32_t)o.arg);
                    put(sums.count == 1   ? Code::kSum1[o.a][sums.axis[0]]
                        : sums.count == 2 ? Code::kSum2[o.a][sums.axis[0]]
                                          : Code::kSum3[o.a],
                        0);
                } else {
                    put(rows == Rows::replace ? (o.c ? Code::kGShift : Code::kUShift)[o.a]
                        : rows == Rows::turn  ? Code::kUTurn[o.a]
                                              : (o.c ? Code::kG : Code::kU)[o.a],
                        (uint32_t)o.arg);
                }
                if (scaled && (*groups)[group_of(o.arg) + 1] == o.arg + 1) {
                    put(Code::kScale, 0);
                    ++dp.n_mats;
                }
                break;
            case OP_TURN:
                if (o.a > 3) return false;
                if constexpr (pair) return false;
                else put(Code::kTurn[o.a], (uint32_t)o.arg);
                break;
            case OP_CX_REG:
                if (o.a > 3 || o.b > 3 || o.a == o.b) return false;
                put(Code::kCx[o.a][o.b], 0);
                break;
            case OP_CX_CHAIN:
                if (o.arg < 0 || o.arg >= (int)(sizeof Code::kChain / sizeof Code::kChain[0])) return false;
                put(Code::kChain[o.arg], 0);
                break;
            case OP_CX_DYN:
                if (o.a > 3 || o.b > 31) return false;
                put(Code::kCxBit[o.a], 1u << o.b);
                break;
            case OP_CX_PAR:
                if (o.a > 3) return false;
                put(Code::kCxParity[o.a], (uint32_t)o.arg);
                break;
            case OP_CX_LANE:
                if (o.a > 3 || o.b > 5) return false;
                if (o.b < 2) put(Code::kCxQuad[o.a][o.b], 0);
                else put(Code::kCxLane[o.a], 1u << o.b);
                break;
            case OP_CZ_MIX:
                if (o.a > 3 || o.b > 31) return false;
                put(Code::kCzMix[o.a], 1u << o.b);
                break;
            case OP_CZ_LANE:
                put(Code::kCzLane, (uint32_t)o.arg);
                break;
            case OP_XPOSE:
                if (s < 0 || s > 10 || o.a > 10) return false;
                put(Code::kWrite[s], Code::kRead[o.a] / 64u | (o.b ? 1u << 16 : 0u) | (o.c ? 1u << 17 : 0u));
                s = o.a;
                break;
            case OP_END:
                put(Code::kEnd, 0);
                break;
            default:
                return false;
        }
    }
    dp.s_out = s;
    if (dp.first_u < 0) dp.first_mat = dp.first_u = 0;
    dp.n_ops = (int)out->ops.size() - dp.begin;
    out->passes.push_back(dp);
    return s >= 0 && !out->ops.empty() && out->ops.back().code == Code::kEnd;
}

inline bool lower_pass(const Op* ops, int count, DirectPlan* out) {
    return lower_pass_as<direct>(ops, count, Rows::none, SumAxes(), nullptr, out);
}

// sums: a mirrored plan for the paired interpreter, which takes the transition sums of its unitaries on the way.
inline bool lower_plan(const Plan& p, Rows rows, DirectPlan* out, const SumAxes* sums = nullptr) {
    for (const Pass& ps : p.passes) {
        if (ps.w + ps.t - ps.c > p.n) return false;
        const Op* ops = p.ops.data() + ps.op_begin;
        if (!(sums ? lower_pass_as<paired>(ops, ps.op_count, Rows::none, *sums, &p.groups, out)
                   : lower_pass_as<direct>(ops, ps.op_count, rows, SumAxes(), &p.groups, out)))
            return false;
        // the table is read front to back
        int next = out->passes.back().first_u;
        for (int k = 0; k < ps.op_count; ++k) {
            const Op& o = p.ops[ps.op_begin + k];
            if (o.kind == OP_U && o.arg != next++) return false;
        }
    }
    return true;
}

}  // namespace qsv
