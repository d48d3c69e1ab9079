"""The direct gate interpreter of the pass kernel, executed instruction by instruction on the CPU: a small
emulator runs the generated text for all lanes of a workgroup at once and the result is compared with the
gates applied to the tile as an array."""
import re

import numpy as np
import pytest

from paper_2602_13140_amd.csrc import gen_gate_asm as g

OFF, END = g.direct_layout()


def _parse():
    """[(byte offset, line)] with the offsets that the sizes and the .org lines give, and the labels."""
    pos, code, labels = 0, [], {}
    for ln in g.gen_direct():
        if ln.startswith(".p2align"):
            continue
        m = re.fullmatch(r"\.org L_dbase_%=\+(\d+), 0", ln)
        if m:
            assert int(m.group(1)) >= pos, ln           # nothing overruns its place
            pos = int(m.group(1))
        elif ln.endswith(":"):
            labels[ln[:-1]] = pos
        else:
            code.append((pos, ln))
            pos += g.size_of(ln)
    return code, labels


CODE, LABELS = _parse()
AT = {pos: i for i, (pos, _) in enumerate(CODE)}


class Machine:
    """State of one workgroup.  Registers are per-lane arrays of 32-bit words, kept as float64 values for
    amplitudes and table entries and as uint32 for the rest."""

    def __init__(self, T, s, tile, c=4, w=6, base=0, ovrid=-1, ovr=None, mats=None, first=0):
        self.T, self.n = T, 1 << (T - g.R)
        thr = np.arange(self.n, dtype=np.uint32)
        tau = lane_tau(T, s)
        self.v = {"thr": thr, "ldsb": (g.padded(tau) * 4).astype(np.uint32),
                  "e0": (expand(tau, c, w) | base).astype(np.uint32)}
        for k in range(16):
            self.v["r%d" % k], self.v["i%d" % k] = tile[tau | (k << s)].real.copy(), tile[tau | (k << s)].imag.copy()
        self.ops = {"c": c, "w": w, "cmask": (1 << c) - 1, "tb": base, "ovrid": ovrid & 0xffffffff, "first": first * 32}
        self.mats, self.ovr = mats, ovr
        self.lds = np.full(1 << 15, np.nan)
        self.s = {}
        self.exec = np.ones(self.n, bool)
        self.steps = 0

    def get(self, tok):
        neg = tok.startswith("-")
        tok = tok.lstrip("-")
        m = re.fullmatch(r"%\[(\w+)\]", tok)
        if m:
            x = self.v[m.group(1)] if m.group(1) in self.v else self.ops[m.group(1)]
        elif tok == "vcc":
            x = self.vcc
        elif tok[0] == "s":
            x = self.s[int(tok[1:])]
        else:
            x = int(tok, 0)
        return -x if neg else x

    def put(self, tok, x):
        name = re.fullmatch(r"%\[(\w+)\]", tok).group(1)
        x = np.broadcast_to(np.asarray(x), self.n).copy()
        if name in self.v and not self.exec.all():
            old = self.v[name]
            x = np.where(self.exec, x, old)
        self.v[name] = x

    def run(self, words):
        pc, scc = 0, 0
        s = self.s
        while True:
            self.steps += 1
            assert self.steps < 200000
            if pc == END:
                return
            pos, ln = CODE[AT[pc]]
            pc += g.size_of(ln)
            op, _, rest = ln.partition(" ")
            a = [t.strip() for t in re.split(r",(?![^\[]*\])", rest)]
            u = lambda i: np.asarray(self.get(a[i])).astype(np.uint64)
            w = lambda x: (x & 0xffffffff).astype(np.uint32)
            if op == "s_getpc_b64":
                s[36], s[37] = pc, 0
            elif op == "s_mov_b64":
                if a[0] == "exec":
                    self.exec = self.saved
            elif op in ("s_add_u32", "s_addc_u32", "s_sub_u32", "s_subb_u32"):
                x, y = int(self.get(a[1])), int(self.get(a[2]))
                x = x + y if "add" in op else x - y
                if op == "s_addc_u32":
                    x += scc
                if op == "s_subb_u32":
                    x -= scc
                scc = int(not 0 <= x <= 0xffffffff)
                s[int(a[0][1:])] = x & 0xffffffff
            elif op == "s_mov_b32":
                s[int(a[0][1:])] = int(self.get(a[1]))
            elif op == "s_and_b32":
                s[int(a[0][1:])] = int(self.get(a[1])) & int(self.get(a[2]))
            elif op == "s_lshl_b32":
                s[int(a[0][1:])] = (int(self.get(a[1])) << int(a[2])) & 0xffffffff
            elif op == "s_load_dwordx2":
                off = 0 if a[2] == "0x0" else s[40]
                s[42], s[43] = words[off // 8]
            elif op == "s_load_dwordx8":
                row, at = (self.ovr, 56) if "ovr" in a[1] else (None, 48)
                if row is None:
                    k = s[41] // 32
                    row = self.mats[k] if k < len(self.mats) else [0.0] * 8
                for k in range(8):
                    s[at + k] = row[k]
            elif op == "s_setpc_b64":
                lo = int(re.match(r"s\[(\d+):", a[0]).group(1))
                assert s[lo + 1] == 0
                pc = s[lo]
            elif op == "s_cmp_eq_u32":
                scc = int(int(self.get(a[0])) == int(self.get(a[1])))
            elif op == "s_bitcmp1_b32":
                scc = (int(self.get(a[0])) >> int(a[1])) & 1
            elif op == "s_branch" or (op == "s_cbranch_scc1" and scc) or (op == "s_cbranch_scc0" and not scc) or \
                    (op == "s_cbranch_execz" and not self.exec.any()):
                pc = LABELS[a[0]]
            elif op in ("s_waitcnt", "s_barrier", "s_cbranch_scc0", "s_cbranch_scc1", "s_cbranch_execz"):
                pass
            elif op == "s_and_saveexec_b64":
                self.saved = self.exec
                self.exec = self.exec & self.vcc
            elif op == "v_fma_f32":
                self.put(a[0], self.get(a[1]) * self.get(a[2]) + self.get(a[3]))
            elif op == "v_fmac_f32":
                self.put(a[0], self.get(a[1]) * self.get(a[2]) + self.get(a[0]))
            elif op == "v_mul_f32":
                self.put(a[0], self.get(a[1]) * self.get(a[2]))
            elif op == "v_mov_b32":
                self.put(a[0], self.get(a[1]))
            elif op == "v_mov_b32_dpp":
                q = [int(x) for x in re.search(r"quad_perm:\[([\d,]+)\]", ln).group(1).split(",")]
                x = self.get(a[1].split()[0])
                lane = np.arange(self.n)
                self.put(a[0], x[(lane & ~3) | np.array(q)[lane & 3]])
            elif op == "ds_bpermute_b32":
                lane = np.arange(self.n)
                self.put(a[0], self.get(a[2])[(lane & ~63) | (self.get(a[1]).astype(int) // 4)])
            elif op == "v_xor_b32" and a[1] == "0x80000000":
                self.put(a[0], -self.get(a[2]))
            elif op == "v_xor_b32":
                self.put(a[0], w(u(1) ^ u(2)))
            elif op == "v_and_b32":
                self.put(a[0], w(u(1) & u(2)))
            elif op == "v_or_b32":
                self.put(a[0], w(u(1) | u(2)))
            elif op == "v_lshrrev_b32":
                self.put(a[0], w(u(2) >> u(1)))
            elif op == "v_lshlrev_b32":
                self.put(a[0], w(u(2) << u(1)))
            elif op == "v_lshl_or_b32":
                self.put(a[0], w((u(1) << u(2)) | u(3)))
            elif op == "v_lshl_add_u32":
                self.put(a[0], w((u(1) << u(2)) + u(3)))
            elif op == "v_bcnt_u32_b32":
                self.put(a[0], np.array([bin(int(x)).count("1") for x in np.broadcast_to(u(1), self.n)], np.uint32))
            elif op == "v_cmp_ne_u32":
                self.vcc = np.asarray(self.get(a[2])) != int(a[1])
            elif op in ("ds_write_b32", "ds_read_b32"):
                off = int(re.search(r"offset:(\d+)", ln).group(1))
                assert off < 65536
                addr = self.get((a[0] if op == "ds_write_b32" else a[1]).split()[0]).astype(int) + off
                assert (addr % 4 == 0).all() and addr.max() < 4 * g.padded(1 << self.T)
                if op == "ds_write_b32":
                    self.lds[addr // 4] = self.get(a[1].split()[0])
                else:
                    self.put(a[0], self.lds[addr // 4])
            else:
                raise AssertionError(ln)

    def tile(self, s):
        out = np.full(1 << self.T, np.nan, complex)
        tau = lane_tau(self.T, s)
        for k in range(16):
            out[tau | (k << s)] = self.v["r%d" % k] + 1j * self.v["i%d" % k]
        return out


def lane_tau(T, s):
    thr = np.arange(1 << (T - g.R))
    return ((thr >> s) << (s + g.R)) | (thr & ((1 << s) - 1))


def expand(tau, c, w):
    return (tau & ((1 << c) - 1)) | ((tau >> c) << w)


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def random_tile(T, seed):
    r = rng(seed)
    return r.standard_normal(1 << T) + 1j * r.standard_normal(1 << T)


def transpose(s, to, cross=1, before=1):
    return (OFF["W%d" % s], OFF["R%d" % to] // 64 | cross << 16 | before << 17)


END_OP = (OFF["END"], 0)


@pytest.mark.parametrize("T", [10, 12, 14])
def test_transposes_between_all_layouts(T):
    t = random_tile(T, T)
    layouts = range(T - 3)
    for s in layouts:
        m = Machine(T, s, t, base=0x5000000, w=7)
        words, at = [], s
        for to in [x for x in layouts for _ in (0, 1)][::3] + [s, 0, T - 4]:
            words.append(transpose(at, to, to & 1, at & 1))
            at = to
        m.mats = []
        m.run(words + [END_OP])
        assert np.array_equal(m.tile(at), t)
        assert np.array_equal(m.v["e0"], expand(lane_tau(T, at), 4, 7) | 0x5000000)


def test_elements_of_a_layout_share_no_bank_between_32_lanes_but_in_the_lowest():
    for s in range(9):
        for half in (0, 32):
            banks = g.padded(lane_tau(12, s)[half:half + 32]) % 32
            assert max(np.bincount(banks, minlength=32)) == (2 if s == 0 else 1), s


def gate(t, bit, m):
    idx = np.arange(t.size)
    lo = idx[(idx >> bit) & 1 == 0]
    a, b = t[lo], t[lo | (1 << bit)]
    t[lo], t[lo | (1 << bit)] = m[0, 0] * a + m[0, 1] * b, m[1, 0] * a + m[1, 1] * b


def factored(r, form, core):
    """A random table entry of a sequence and its matrix."""
    first = r.uniform(-np.pi / 2, np.pi / 2) if form.startswith(("before", "both")) else 0.0
    last = r.uniform(-np.pi / 2, np.pi / 2) if form.startswith(("after", "both")) else 0.0
    x, y = r.uniform(-1, 1, 2)
    sign = -1.0 if g.CORES[core][1] == "-" else 1.0
    k = np.array([[1, x], [y, sign]] if g.CORES[core][0] == "c" else [[x, -sign], [1, y]], dtype=complex)
    e = [-np.tan(first / 2), np.sin(first), x, y, -np.tan(last / 2), np.sin(last), OFF["F%s%d" % (form, core)], 0.0]
    zb, za = np.exp(1j * last) * (1j if "B" in form else 1), np.exp(1j * first) * (1j if "A" in form else 1)
    return e, np.diag([1, zb]) @ k @ np.diag([1, za])


@pytest.mark.parametrize("shifts", [0, 1])
def test_unitaries_of_every_kind(shifts):
    """All sequences on all register bits and whole matrices among them, the table read from entry 3 on; with
    `shifts` one factored and one whole entry are replaced by the row's shifted matrix in turn."""
    T, s = 10, 5
    r = rng(3)
    kinds = [(f, c, j) for f in g.FORMS for c in range(4) for j in range(4)] + [("whole", 0, j) for j in range(4)]
    kinds = [kinds[i] for i in r.permutation(len(kinds))]
    over_m = r.standard_normal(8)
    for over in ([None] if not shifts else [None, 3 + kinds.index(("both", 1, 2)), 3 + kinds.index(("whole", 0, 1))]):
        r = rng(4)
        t = random_tile(T, 9)
        want = t.copy()
        mats, words = [[0.0] * 8] * 3, []
        for f, c, j in kinds:
            k = len(mats)
            if f == "whole":
                e = r.standard_normal(8)
                m = (e[0::2] + 1j * e[1::2]).reshape(2, 2)
                words.append((OFF["%s%d" % ("GS" if shifts else "G", j)], k))
            else:
                e, m = factored(r, f, c)
                words.append((OFF["%s%d" % ("US" if shifts else "U", j)], k))
            mats.append(list(e))
            if k == over:
                m = (over_m[0::2] + 1j * over_m[1::2]).reshape(2, 2)
            gate(want, s + j, m)
        mach = Machine(T, s, t, mats=mats, first=3, ovrid=-1 if over is None else over, ovr=list(over_m))
        mach.run(words + [END_OP])
        assert np.allclose(mach.tile(s), want, rtol=1e-9, atol=1e-9 * np.abs(want).max())


def test_permutations_and_signs():
    """Every CNOT and CZ form, against the same gates on the tile's indices."""
    T, s, c, w = 12, 4, 4, 9
    base = 0x0c00000 & ~expand((1 << T) - 1, c, w) | 0x20
    t = random_tile(T, 5)
    want = t.copy()
    words = []
    tau = np.arange(1 << T)
    e = expand(tau, c, w) | base

    def move(cond, bit):
        src = np.where(cond, tau ^ (1 << bit), tau)
        want[:] = want[src].copy()

    def sign(cond):
        want[cond] = -want[cond]

    bit = lambda x, k: (x >> k) & 1 == 1
    par = lambda x: np.array([bin(int(v)).count("1") & 1 for v in x]) == 1
    for jt in range(4):
        for jc in range(4):
            if jt != jc:
                words.append((OFF["X%d%d" % (jt, jc)], 0))
                move(bit(tau, s + jc), s + jt)
    for k, (d, first, count) in enumerate(g.CX_CHAINS):
        words.append((OFF["C%d" % k], 0))
        for i in range(count):
            cc = first + i if d == 0 else first - i
            move(bit(tau, s + cc), s + cc + 1)
    for j in range(4):
        for q in (0, 3, 13, 16, 23, 22, 5, 8):                  # lane, wavefront and tile bits; bits 23 and 5 are set, 8 is not
            words.append((OFF["D%d" % j], 1 << q))
            move(bit(e, q), s + j)
        mask = 1 << 0 | 1 << 14 | 1 << 22 | 1 << 23
        words.append((OFF["P%d" % j], mask))
        move(par(e & mask), s + j)
    lane_bits = [0, 1, 2, 3, 8, 9]                              # tile bits behind the lane bits in layout 4
    for j in range(4):
        for b in range(6):
            words.append((OFF["N%d%d" % (j, b)], 0) if b < 2 else (OFF["N%d" % j], 1 << b))
            move(bit(tau, s + j), lane_bits[b])
    for m in range(1, 8):
        words.append((OFF["ZR%d" % m], 0))
        run = (tau >> s) & 15
        sign(par(run & (run >> 1) & m))
    for j in range(4):
        for q in (2, 13, 15, 23, 8):
            words.append((OFF["ZM%d" % j], 1 << q))
            sign(bit(tau, s + j) & bit(e, q))
    # rungs between neighbouring index bits of which none is in the run (index bits 9..12)
    mask = 1 << 0 | 1 << 1 | 1 << 13 | 1 << 14 | 1 << 22
    words.append((OFF["ZL"], mask))
    sign(par(e & (e >> 1) & mask))
    m = Machine(T, s, t, c=c, w=w, base=base, mats=[])
    m.run(words + [END_OP])
    assert np.array_equal(m.tile(s), want)


def test_text_uses_its_scalar_registers_only_and_has_every_label_once():
    text = "\n".join(g.gen_direct())
    for m in re.finditer(r"\bs\[?(\d+)(?::(\d+))?", text):
        assert g.DIRECT_FIRST <= int(m.group(1)) and int(m.group(2) or m.group(1)) <= g.DIRECT_LAST
    labels = [ln for ln in g.gen_direct() if ln.endswith(":")]
    assert len(labels) == len(set(labels))
    # every piece of code ends in a jump: nothing runs on into its neighbour
    lines = [ln for ln in g.gen_direct() if not ln.startswith(".p2")]
    for i, ln in enumerate(lines):
        if ln.startswith(".org"):
            assert lines[i - 1].startswith(("s_setpc_b64", "s_branch")), lines[i - 1]


def test_every_operation_fetches_one_word_and_waits_before_it_jumps():
    for name, lines in g.direct_handlers():
        jumps = [i for i, ln in enumerate(lines) if ln == "s_setpc_b64 s[64:65]"]
        if name.startswith(("US", "U", "R")) and not name.startswith("RI"):
            continue                       # a stub, or the middle of a transpose
        fetch = sum(ln == g.NEXT_WORD[1] for ln in lines)
        assert fetch == (0 if name == "END" or name.startswith(("GS", "WI", "RI")) else 1), name
        for i in jumps:
            assert lines[i - 3] == "s_waitcnt lgkmcnt(0)", name
