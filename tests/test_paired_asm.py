"""The paired gate interpreter (two states at once, with transition sums), executed instruction by instruction on
the CPU: every operation must do to both states what the gate does, and every record of sums must be the sum over the
wavefront's pairs of the state as it is at that point."""
import re

import numpy as np
import pytest

from paper_2602_13140_amd.csrc import gen_gate_asm as g
from tests import test_direct_asm as d

OFF, END = g.direct_layout(True)


def _parse():
    pos, code, labels = 0, [], {}
    for ln in g.gen_direct(True):
        if ln.startswith(".p2align"):
            continue
        m = re.fullmatch(r"\.org L_dbase_%=\+(\d+), 0", ln)
        if m:
            assert int(m.group(1)) >= pos, ln            # nothing overruns its place
            pos = int(m.group(1))
        elif ln.endswith(":"):
            assert ln[:-1] not in labels
            labels[ln[:-1]] = pos
        else:
            code.append((pos, ln))
            pos += g.size_of(ln)
    return code, labels


CODE, LABELS = _parse()
AT = {pos: i for i, (pos, _) in enumerate(CODE)}
STEP = 1 << 20                                           # bytes from a unitary's records to the next one's


class Pair:
    """One workgroup with psi in r, i and lambda in p, q."""

    def __init__(self, T, s, psi, lam, c=4, w=6, base=0, mats=(), first=0):
        self.T, self.n = T, 1 << (T - g.R)
        tau = d.lane_tau(T, s)
        thr = np.arange(self.n)
        self.v = {"thr": thr, "ldsb": 4 * g.padded(tau), "e0": d.expand(tau, c, w) | base}
        for k in range(16):
            for x, st in (("r", psi.real), ("i", psi.imag), ("p", lam.real), ("q", lam.imag)):
                self.v["%s%d" % (x, k)] = st[tau | (k << s)].copy()
        self.sc = {"c": c, "w": w, "cmask": (1 << c) - 1, "tb": base, "sstep": STEP, "first": 32 * first}
        self.mats = mats
        self.lds = np.full(1 << 16, np.nan)
        self.records = {}

    def tiles(self, s):
        tau = d.lane_tau(self.T, s)
        out = []
        for re_, im in ("ri", "pq"):
            t = np.full(1 << self.T, np.nan, complex)
            for k in range(16):
                t[tau | (k << s)] = self.v["%s%d" % (re_, k)] + 1j * self.v["%s%d" % (im, k)]
            out.append(t)
        return out

    def run(self, words):
        s, v, n = {}, self.v, self.n
        pc = scc = 0
        ex = np.ones(n, bool)
        saved = vcc = None
        while pc != END:
            pos, ln = CODE[AT[pc]]
            pc += g.size_of(ln)
            op, _, rest = ln.partition(" ")
            a = [t.strip() for t in re.split(r",(?![^\[]*\])", rest)]

            def get(tok):
                tok = tok.split()[0]
                neg, tok = tok.startswith("-%"), tok.lstrip("-") if tok.startswith("-%") else tok
                m = re.fullmatch(r"%\[(\w+)\]", tok)
                x = (v[m.group(1)] if m.group(1) in v else self.sc[m.group(1)]) if m else \
                    s[int(tok[1:])] if re.fullmatch(r"s\d+", tok) else int(tok, 0)
                return -x if neg else x

            def put(tok, x):
                name = re.fullmatch(r"%\[(\w+)\]", tok).group(1)
                x = np.broadcast_to(np.asarray(x), n).copy()
                v[name] = np.where(ex, x, v[name]) if name in v and not ex.all() else x

            i = lambda k: np.asarray(get(a[k])).astype(np.int64)
            w = lambda x: x & 0xffffffff
            if op == "s_getpc_b64":
                s[36], s[37] = pc, 0
            elif op == "s_mov_b64":
                if a[0] == "exec":
                    if a[1] == "s[74:75]":
                        assert s[74] == s[75] == 0x10001
                        ex = np.arange(n) % 16 == 0
                    else:
                        ex = np.ones(n, bool) if a[1] == "-1" else saved
                elif a[0] == "s[72:73]":
                    s[72], s[73] = 0, 0
            elif op in ("s_add_u32", "s_addc_u32", "s_sub_u32", "s_subb_u32"):
                x = int(get(a[1])) + (int(get(a[2])) if "add" in op else -int(get(a[2])))
                x += scc if op == "s_addc_u32" else -scc if op == "s_subb_u32" else 0
                scc = int(not 0 <= x <= 0xffffffff)
                s[int(a[0][1:])] = x & 0xffffffff
            elif op == "s_mov_b32":
                s[int(a[0][1:])] = int(get(a[1]))
            elif op == "s_and_b32":
                s[int(a[0][1:])] = int(get(a[1])) & int(get(a[2]))
            elif op == "s_lshl_b32":
                s[int(a[0][1:])] = (int(get(a[1])) << int(a[2])) & 0xffffffff
            elif op == "s_load_dwordx2":
                s[42], s[43] = words[(0 if a[2] == "0x0" else s[40]) // 8]
            elif op == "s_load_dwordx8":
                row = self.mats[s[41] // 32] if s[41] // 32 < len(self.mats) else [0.0] * 8
                for k in range(8):
                    s[48 + k] = row[k]
            elif op == "s_setpc_b64":
                lo = int(re.match(r"s\[(\d+):", a[0]).group(1))
                assert s[lo + 1] == 0
                pc = s[lo]
            elif op == "s_bitcmp1_b32":
                scc = (int(get(a[0])) >> int(a[1])) & 1
            elif op == "s_branch" or (op == "s_cbranch_scc0" and not scc) or (op == "s_cbranch_execz" and not ex.any()):
                pc = LABELS[a[0]]
            elif op in ("s_waitcnt", "s_barrier", "s_nop", "s_cbranch_scc0", "s_cbranch_execz"):
                pass
            elif op == "s_and_saveexec_b64":
                saved, ex = ex, ex & vcc
            elif op == "v_fma_f32":
                put(a[0], get(a[1]) * get(a[2]) + get(a[3]))
            elif op == "v_fmac_f32":
                put(a[0], get(a[1]) * get(a[2]) + get(a[0]))
            elif op == "v_mul_f32":
                put(a[0], get(a[1]) * get(a[2]))
            elif op == "v_add_f32":
                put(a[0], get(a[1]) + get(a[2]))
            elif op == "v_mov_b32":
                put(a[0], get(a[1]))
            elif op in ("v_mov_b32_dpp", "v_add_f32_dpp"):
                x, lane = get(a[1]), np.arange(n)
                m = re.search(r"quad_perm:\[([\d,]+)\]", ln)
                if m:
                    src = (lane & ~3) | np.array([int(q) for q in m.group(1).split(",")])[lane & 3]
                else:
                    src = (lane & ~15) | ((lane - int(re.search(r"row_ror:(\d+)", ln).group(1))) & 15)
                put(a[0], x[src] if op == "v_mov_b32_dpp" else x[src] + get(a[2]))
            elif op in ("v_permlane32_swap_b32", "v_permlane16_swap_b32"):
                half = 32 if "32" in op[:14] else 16      # the upper halves of one, the lower halves of the other
                x, y, lane = get(a[0]).copy(), get(a[1]).copy(), np.arange(n)
                up = (lane & half) != 0
                put(a[0], np.where(up, y[lane ^ half], x))
                put(a[1], np.where(up, y, x[lane ^ half]))
            elif op == "global_store_dword":
                addr, x = get(a[0]) + s[72] + (s[73] << 32), get(a[1])
                for k in np.nonzero(ex)[0]:
                    assert int(addr[k]) not in self.records
                    self.records[int(addr[k])] = x[k]
            elif op == "ds_bpermute_b32":
                put(a[0], get(a[2])[(np.arange(n) & ~63) | (get(a[1]) // 4)])
            elif op == "v_xor_b32" and a[1] == "0x80000000":
                put(a[0], -get(a[2]))
            elif op == "v_xor_b32":
                put(a[0], w(i(1) ^ i(2)))
            elif op == "v_and_b32":
                put(a[0], w(i(1) & i(2)))
            elif op == "v_or_b32":
                put(a[0], w(i(1) | i(2)))
            elif op == "v_add_u32":
                put(a[0], w(i(1) + i(2)))
            elif op == "v_lshrrev_b32":
                put(a[0], w(i(2) >> i(1)))
            elif op == "v_lshlrev_b32":
                put(a[0], w(i(2) << i(1)))
            elif op == "v_lshl_or_b32":
                put(a[0], w((i(1) << i(2)) | i(3)))
            elif op == "v_lshl_add_u32":
                put(a[0], w((i(1) << i(2)) + i(3)))
            elif op == "v_bcnt_u32_b32":
                put(a[0], np.array([bin(int(x)).count("1") for x in np.broadcast_to(i(1), n)]))
            elif op == "v_cmp_ne_u32":
                vcc = np.asarray(get(a[2])) != int(a[1])
            elif op in ("ds_write_b32", "ds_read_b32"):
                off = int(re.search(r"offset:(\d+)", ln).group(1))
                assert off < 65536
                addr = get(a[0] if op == "ds_write_b32" else a[1]).astype(int) + off
                assert (addr % 4 == 0).all() and addr.max() < 4 * g.padded(1 << self.T)
                if op == "ds_write_b32":
                    self.lds[addr // 4] = get(a[1])
                else:
                    put(a[0], self.lds[addr // 4])
            else:
                raise AssertionError(ln)


def two_tiles(T, seed):
    return d.random_tile(T, seed), d.random_tile(T, seed + 100)


def transpose(s, to, cross=1, before=1):
    return (OFF["W%d" % s], OFF["R%d" % to] // 64 | cross << 16 | before << 17)


END_OP = (OFF["END"], 0)
PAULI = {"X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.diag([1, -1])}


@pytest.mark.parametrize("T", [10, 13])
def test_transposes_between_all_layouts(T):
    psi, lam = two_tiles(T, T)
    for s in range(T - 3):
        m = Pair(T, s, psi, lam, base=0x5000000, w=7)
        words, at = [], s
        for to in [x for x in range(T - 3) for _ in (0, 1)][::3] + [s, 0, T - 4]:
            words.append(transpose(at, to, to & 1, at & 1))
            at = to
        m.run(words + [END_OP])
        for got, want in zip(m.tiles(at), (psi, lam)):
            assert np.array_equal(got, want)
        assert np.array_equal(m.v["e0"], d.expand(d.lane_tau(T, at), 4, 7) | 0x5000000)


def wavefront_sums(T, s, psi, lam, bit, axis):
    """Im <lambda| P |psi> over each wavefront's amplitudes."""
    phi = psi.copy()
    d.gate(phi, bit, PAULI[axis])
    t = (lam.conj() * phi).imag
    tau = d.lane_tau(T, s)
    return sum(t[tau | (k << s)] for k in range(16)).reshape(-1, 64).sum(1)


def test_unitaries_of_every_kind_and_the_sums_around_them():
    """All sequences on all register bits, scalars among them, on both states, with every kind of sums in turn."""
    T, s = 11, 5
    r = d.rng(3)
    kinds = [(f, c, j) for f in g.FORMS for c in range(4) for j in range(4)] + [("scale", 0, j) for j in range(4)]
    kinds = [kinds[i] for i in r.permutation(len(kinds))]
    psi, lam = two_tiles(T, 9)
    want = [psi.copy(), lam.copy()]
    mats, words, records = [[0.0] * 8] * 3, [], []
    for nth, (f, c, j) in enumerate(kinds):
        if f == "scale":
            e = r.standard_normal(8) / 2
            m = (e[0] + 1j * e[1]) * np.eye(2)
        else:
            e, m = d.factored(r, f, c)
            e[6] = OFF["F%s%d" % (f, c)]
        how, axis, first = nth % 3 + 1, "XYZ"[nth // 3 % 3], "XYZ"[nth // 9 % 3]
        sums = lambda x: wavefront_sums(T, s, want[0], want[1], s + j, x)
        if how == 2:
            words.append((OFF["B%d%s" % (j, first)], 0))
            before = sums(first)
        words.append((OFF["M" if f == "scale" else "U%d" % j], len(mats)))
        mats.append(list(e))
        for t in want:
            d.gate(t, s + j, m)
        words.append((OFF["S3%d" % j if how == 3 else "S%d%d%s" % (how, j, axis)], 0))
        records.append([sums("X"), sums("Z"), sums("Y"), 0 * sums("Y")] if how == 3 else
                       [sums(axis)] * 2 + [before if how == 2 else sums(axis)] * 2)
    mach = Pair(T, s, psi, lam, mats=mats, first=3)
    mach.run(words + [END_OP])
    for got, t in zip(mach.tiles(s), want):
        assert np.allclose(got, t, rtol=1e-9, atol=1e-9 * np.abs(t).max())
    assert len(mach.records) == 4 * (mach.n // 64) * len(records)
    for u, rec in enumerate(records):
        for x, per_wave in enumerate(rec):
            for wv, value in enumerate(per_wave):
                got = mach.records[u * STEP + wv * 16 + x * 4]
                assert abs(got - value) <= 1e-9 * (np.abs(want[0]).max() * np.abs(want[1]).max() * 2048 + abs(value)), (u, x, wv)


def test_permutations_and_signs():
    """Every CNOT and CZ form does to both states what it does to one in the direct interpreter."""
    T, s, c, w = 12, 4, 4, 9
    base = 0x0c00000 & ~d.expand((1 << T) - 1, c, w) | 0x20
    psi, lam = two_tiles(T, 5)
    names = [("X%d%d" % (t, k), 0) for t in range(4) for k in range(4) if t != k]
    names += [("C%d" % k, 0) for k in range(len(g.CX_CHAINS))]
    names += [("D%d" % j, 1 << q) for j in range(4) for q in (0, 3, 13, 23, 5, 8)]
    names += [("P%d" % j, 1 << 0 | 1 << 14 | 1 << 22 | 1 << 23) for j in range(4)]
    names += [("N%d%d" % (j, b), 0) for j in range(4) for b in (0, 1)]
    names += [("N%d" % j, 1 << b) for j in range(4) for b in range(2, 6)]
    names += [("ZR%d" % m, 0) for m in range(1, 8)] + [("ZM%d" % j, 1 << q) for j in range(4) for q in (2, 13, 23)]
    names += [("ZL", 1 << 0 | 1 << 1 | 1 << 13 | 1 << 14 | 1 << 22)]
    pair = Pair(T, s, psi, lam, c=c, w=w, base=base)
    pair.run([(OFF[k], x) for k, x in names] + [END_OP])
    for got, t in zip(pair.tiles(s), (psi, lam)):
        one = d.Machine(T, s, t, c=c, w=w, base=base, mats=[])
        one.run([(d.OFF[k], x) for k, x in names] + [d.END_OP])
        assert np.array_equal(got, one.tile(s))


def test_text_uses_its_scalar_registers_only_and_waits_before_it_jumps():
    text = "\n".join(g.gen_direct(True))
    for m in re.finditer(r"\bs\[?(\d+)(?::(\d+))?", text):
        assert g.DIRECT_FIRST <= int(m.group(1)) and int(m.group(2) or m.group(1)) <= g.PAIR_LAST
    lines = [ln for ln in g.gen_direct(True) if not ln.startswith(".p2")]
    for i, ln in enumerate(lines):
        if ln.startswith(".org"):
            assert lines[i - 1].startswith(("s_setpc_b64", "s_branch")), lines[i - 1]
    for name, ls in g.direct_handlers(True):
        if name.startswith("U") or name.startswith("R") and not name.startswith("RLI"):
            continue                       # a stub, or the middle of a transpose
        assert sum(ln == g.NEXT_WORD[1] for ln in ls) == (0 if name.startswith(("END", "WI", "WL", "RI", "RL")) else 1), name
        for i, ln in enumerate(ls):
            if ln == "s_setpc_b64 s[64:65]":
                assert ls[i - 3] == "s_waitcnt lgkmcnt(0)", name
            if "permlane" in ln or ln.startswith("v_add_f32_dpp"):
                assert ls[i - 1] == "s_nop 1", name     # two wait states after a write of the register
