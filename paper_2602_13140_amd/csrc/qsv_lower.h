// Operation lists of a plan in the form that the direct interpreter of the pass kernel reads.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "qsv_gate_asm.h"
#include "qsv_plan.h"

namespace qsv {

struct DirectOp {
    uint32_t code;   // byte offset of the operation's code in the interpreter
    uint32_t arg;    // unitaries: index in execution order; conditions: mask of index bits; lane exchange: mask of the
                     // lane number; transposes: offset / 64 of the target layout's code | flags << 16
};
static_assert(sizeof(DirectOp) == sizeof(Op), "both forms take the same room");

struct DirectPass {
    int begin;           // first operation
    int s_in, s_out;     // register layouts of the load and the store
    int first_mat;       // index of the first unitary (0 if none)
};

struct DirectPlan {
    std::vector<DirectOp> ops;   // never more than the plan has
    std::vector<DirectPass> passes;
};

// Lowers one operation list (a pass: OP_LOAD ... OP_END) onto out; false if it holds something the direct
// interpreter has no code for (never planned for tiles of one row).  shifts: some row may replace a matrix.
inline bool lower_pass(const Op* ops, int count, bool shifts, DirectPlan* out) {
    DirectPass dp;
    dp.begin = (int)out->ops.size();
    dp.s_in = dp.s_out = -1;
    dp.first_mat = -1;
    int s = -1;
    uint32_t rungs = 0;          // CZ rungs inside the run, collected: neighbouring ones go in one operation
    auto put = [&](uint32_t code, uint32_t arg) { out->ops.push_back({code, arg}); };
    auto flush = [&]() {
        if (rungs) put(direct::kCz[rungs], 0);
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
                if (dp.first_mat < 0) dp.first_mat = o.arg;
                put(o.c ? (shifts ? direct::kGShift[o.a] : direct::kG[o.a]) : (shifts ? direct::kUShift[o.a] : direct::kU[o.a]),
                    (uint32_t)o.arg);
                break;
            case OP_CX_REG:
                if (o.a > 3 || o.b > 3 || o.a == o.b) return false;
                put(direct::kCx[o.a][o.b], 0);
                break;
            case OP_CX_CHAIN:
                if (o.arg < 0 || o.arg >= (int)(sizeof direct::kChain / sizeof direct::kChain[0])) return false;
                put(direct::kChain[o.arg], 0);
                break;
            case OP_CX_DYN:
                if (o.a > 3 || o.b > 31) return false;
                put(direct::kCxBit[o.a], 1u << o.b);
                break;
            case OP_CX_PAR:
                if (o.a > 3) return false;
                put(direct::kCxParity[o.a], (uint32_t)o.arg);
                break;
            case OP_CX_LANE:
                if (o.a > 3 || o.b > 5) return false;
                if (o.b < 2) put(direct::kCxQuad[o.a][o.b], 0);
                else put(direct::kCxLane[o.a], 1u << o.b);
                break;
            case OP_CZ_MIX:
                if (o.a > 3 || o.b > 31) return false;
                put(direct::kCzMix[o.a], 1u << o.b);
                break;
            case OP_CZ_LANE:
                put(direct::kCzLane, (uint32_t)o.arg);
                break;
            case OP_XPOSE:
                if (s < 0 || s > 10 || o.a > 10) return false;
                put(direct::kWrite[s], direct::kRead[o.a] / 64u | (o.b ? 1u << 16 : 0u) | (o.c ? 1u << 17 : 0u));
                s = o.a;
                break;
            case OP_END:
                put(direct::kEnd, 0);
                break;
            default:
                return false;
        }
    }
    dp.s_out = s;
    if (dp.first_mat < 0) dp.first_mat = 0;
    out->passes.push_back(dp);
    return s >= 0 && !out->ops.empty() && out->ops.back().code == direct::kEnd;
}

inline bool lower_plan(const Plan& p, bool shifts, DirectPlan* out) {
    for (const Pass& ps : p.passes) {
        if (ps.w + ps.t - ps.c > p.n) return false;
        if (!lower_pass(p.ops.data() + ps.op_begin, ps.op_count, shifts, out)) return false;
        // the table is read front to back
        int next = out->passes.back().first_mat;
        for (int k = 0; k < ps.op_count; ++k) {
            const Op& o = p.ops[ps.op_begin + k];
            if (o.kind == OP_U && o.arg != next++) return false;
        }
    }
    return true;
}

}  // namespace qsv
