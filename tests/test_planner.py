"""Host-logic tests (no GPU): the pass planner's operation lists, replayed by a small numpy
interpreter that follows the documented meaning of each operation, must reproduce the oracle's
circuit.  This checks the lowering, the commutation rules and the tile/run bookkeeping before any
kernel runs."""
import ctypes

import numpy as np
import pytest

from paper_2602_13140_amd import binding as qb
from tests import dense_bruteforce as dense

RX, RY, RZ = 1, 2, 3
NONE, RING, LADDER = 0, 1, 2
R = 4


def parse_plan(text):
    lines = text.strip().split("\n")
    head = dict(kv.split("=") for kv in lines[0].split()[1:])
    passes = []
    for ln in lines[1:]:
        hdr, ops = ln.split(":", 1)
        kv = dict(x.split("=") for x in hdr.split()[1:])
        passes.append(({k: int(v) for k, v in kv.items()}, ops.split()))
    return {k: int(v) for k, v in head.items()}, passes


def fused_matrix(rot, reupload, layer_params, feat_q, q, inverse):
    """U(l,q) = R_last ... R_first (re-upload RX first); dagger in inverse mode."""
    u = np.eye(2, dtype=np.complex128)
    slot = 0
    if reupload:
        u = dense.rot_matrix(RX, layer_params[0][q] * feat_q) @ u
        slot = 1
    for r, axis in enumerate(rot):
        u = dense.rot_matrix(axis, layer_params[slot + r][q]) @ u
    return u.conj().T if inverse else u


def apply_1q(st, n, q, mats):
    """st: [rows, 2^n]; mats: [rows, 2, 2] or [2, 2]."""
    rows = st.shape[0]
    v = st.reshape(rows, 1 << (n - 1 - q), 2, 1 << q)
    if mats.ndim == 2:
        out = np.einsum("ab,rhbl->rhal", mats, v)
    else:
        out = np.einsum("rab,rhbl->rhal", mats, v)
    return out.reshape(rows, 1 << n)


def apply_cnot(st, n, ctrl, tgt):
    k = np.arange(1 << n)
    src = np.where((k >> ctrl) & 1, k ^ (1 << tgt), k)
    return st[:, src]


def apply_index_map(st, n, imap):
    """What a pass with deferred CNOTs does when it stores: the amplitude at position p goes to the
    index that is the XOR of imap[j] over the set bits j of p."""
    assert len(imap) == n
    k = np.arange(1 << n)
    dest = np.zeros(1 << n, dtype=np.int64)
    for j in range(n):
        assert (imap[j] >> j) & 1                    # a position bit always maps onto itself as well
        if j < 3:
            assert imap[j] == 1 << j                 # runs of 64 bytes are written whole
        dest ^= np.where((k >> j) & 1, imap[j], 0)
    assert len(np.unique(dest)) == 1 << n            # a permutation
    out = np.empty_like(st)
    out[:, dest] = st
    return out


def apply_parity_cnot(st, n, mask, tgt):
    k = np.arange(1 << n)
    par = np.zeros(1 << n, dtype=np.int64)
    for j in range(n):
        if (mask >> j) & 1:
            par ^= (k >> j) & 1
    src = np.where(par == 1, k ^ (1 << tgt), k)
    return st[:, src]


def replay(text, n, rows, L, rot, ent, reupload, params, feats, inverse, st):
    """Within a pass, `st` is indexed by position (where the amplitude sits: the kernel's view); passes
    without deferred CNOTs never tell the difference."""
    head, passes = parse_plan(text)
    assert head["n"] == n
    slots = int(reupload) + len(rot)
    p = np.asarray(params, dtype=np.float64).reshape(L, slots, n)
    n_gates = 0
    for hdr, ops in passes:
        t, c, w = hdr["t"], hdr["c"], hdr["w"]
        assert 10 <= t <= 14 and 3 <= c <= t and w >= c
        bit = lambda pos: pos if pos < c else pos - c + w
        if n > t:
            assert w + (t - c) <= n
        assert ops[0][0] == "L" and "E" in ops
        tail = ops[ops.index("E") + 1:]
        assert all(tk[0] in "VM" for tk in tail)          # after the store: the deferred CNOTs and the map
        local_bits = [bit(pp) for pp in range(t)]
        s = None
        for tok in ops:
            kind = tok[0]
            if kind in "LT":
                s_prev = s
                s = int(tok[1:].split(":")[0])
                assert 0 <= s <= t - R
                if kind == "L":
                    assert s >= min(4, t - R)
                    seen_xpose, prev_cross = False, False
                else:
                    # barrier flags: bit 0 = exchange crosses wavefronts, bit 1 = barrier first
                    flags = int(tok.split(":")[1])
                    cross = s_prev + R > 10 or s + R > 10
                    assert (flags & 1) == int(cross)
                    assert (flags >> 1) == int(seen_xpose and (cross or prev_cross))
                    seen_xpose, prev_cross = True, cross
            elif kind == "U":
                j, mat, rowdep = (int(x) for x in tok[1:].split(":"))
                q = bit(s + j)
                assert q < n and 0 <= j < R
                l = mat // n
                assert mat % n == q
                if reupload:
                    assert rowdep == 1
                    if n < t:
                        assert s + R <= n      # a lane's 16 amplitudes share one row
                    ms = np.stack([fused_matrix(rot, 1, p[l], feats[r][q], q, inverse)
                                   for r in range(rows)])
                else:
                    ms = fused_matrix(rot, 0, p[l], None, q, inverse)
                st = apply_1q(st, n, q, ms)
                n_gates += 1
            elif kind == "X":
                jt, jc = (int(x) for x in tok[1:].split(":"))
                assert jt != jc
                st = apply_cnot(st, n, bit(s + jc), bit(s + jt))
                n_gates += 1
            elif kind == "C":
                # chain of CNOTs between neighbouring register bits: "u": a->a+1, a+1->a+2, ...;
                # "d": a->a+1, a-1->a, ...
                jc, count = (int(x) for x in tok[2:].split(":"))
                assert tok[1] in "ud" and count in (2, 3)
                for i in range(count):
                    c0 = jc + i if tok[1] == "u" else jc - i
                    assert 0 <= c0 and c0 + 1 < R
                    st = apply_cnot(st, n, bit(s + c0), bit(s + c0 + 1))
                    n_gates += 1
            elif kind == "D":
                jt, qc, uni = (int(x) for x in tok[1:].split(":"))
                qt = bit(s + jt)
                assert qt < n and qc < n and qc != qt
                run_bits = [bit(s + j) for j in range(R)]
                assert qc not in run_bits
                local = [bit(pp) for pp in range(t)]
                if qc in local:
                    pc = local.index(qc)
                    tbit = pc if pc < s else pc - R
                    assert uni == (1 if tbit >= 6 else 0)
                else:
                    assert uni == 1
                st = apply_cnot(st, n, qc, qt)
                n_gates += 1
            elif kind == "N":
                # CNOT with the control in register bit jc and the target behind bit b of the lane number
                jc, b, qt = (int(x) for x in tok[1:].split(":"))
                run_bits = [bit(s + j) for j in range(R)]
                assert 0 <= jc < R and qt not in run_bits and qt in local_bits and 0 <= b < 6
                pp = local_bits.index(qt)
                assert b == (pp if pp < s else pp - R)        # where the lane number keeps that tile bit
                st = apply_cnot(st, n, run_bits[jc], qt)
                n_gates += 1
            elif kind == "Q":
                # CNOT on register bit jt under the parity of the position bits in mask
                jt, qc, mask = tok[1:].split(":")
                jt, qc, mask = int(jt), int(qc), int(mask, 16)
                qt = bit(s + jt)
                run_bits = [bit(s + j) for j in range(R)]
                assert qt < n and mask < (1 << n) and bin(mask).count("1") >= 2
                assert not any((mask >> q) & 1 for q in run_bits)
                st = apply_parity_cnot(st, n, mask, qt)
                n_gates += 1
            elif kind == "V":
                # deferred CNOT: target outside the tile, carried by the map; nothing moves now
                qt, qc, mask = tok[1:].split(":")
                qt, qc, mask = int(qt), int(qc), int(mask, 16)
                assert qt not in local_bits and qt < n and not (mask & 7) and not (mask >> qt) & 1
                n_gates += 1
            elif kind == "M":
                st = apply_index_map(st, n, [int(x, 16) for x in tok[1:].split(",")])
            elif kind == "Z":
                form, body = tok[1], tok[2:]
                run_bits = [bit(s + j) for j in range(R)]
                if form == "r":                       # both qubits in the register run
                    ja, jb = (int(x) for x in body.split(":"))
                    assert 0 <= ja < jb < R
                    rungs = [(run_bits[ja], run_bits[jb])]
                elif form == "m":                     # one in the run, one elsewhere
                    ja, qo = (int(x) for x in body.split(":"))
                    assert qo not in run_bits and qo < n
                    rungs = [(run_bits[ja], qo)]
                else:                                 # mask of rungs (q, q+1), none in the run
                    assert form == "l"
                    mask = int(body, 16)
                    rungs = [(q, q + 1) for q in range(n) if (mask >> q) & 1]
                    assert all(q0 not in run_bits and q1 not in run_bits for q0, q1 in rungs)
                k = np.arange(1 << n)
                for q0, q1 in rungs:
                    assert abs(q0 - q1) == 1 and max(q0, q1) < n       # a ladder rung
                    st = st * (1 - 2 * (((k >> q0) & 1) & ((k >> q1) & 1)))[None, :]
                    n_gates += 1
            else:
                assert tok == "E"
        assert sum(1 for o in ops if o == "E") == 1
        assert sum(1 for o in ops if o[0] == "V") == 0 or sum(1 for o in ops if o[0] == "M") == 1
    return st, n_gates, len(passes)


CASES = [
    # n, rows, L, rot, ent, reupload, tile
    (4, 8, 2, (RY, RZ), RING, 0, 0), (5, 3, 3, (RX, RY, RZ), RING, 0, 0),
    (7, 2, 2, (RY, RZ), LADDER, 0, 0), (6, 5, 3, (RY, RZ), RING, 1, 0),
    (10, 2, 3, (RY, RZ), RING, 1, 0), (11, 1, 3, (RX, RY, RZ), RING, 0, 10),
    (12, 1, 2, (RY, RZ), LADDER, 0, 10), (12, 2, 3, (RY, RZ), RING, 0, 11),
    (13, 1, 3, (RY, RZ), RING, 0, 10), (13, 1, 2, (RX,), NONE, 0, 12),
    (12, 1, 2, (), RING, 0, 10), (12, 2, 2, (RY, RZ), RING, 1, 10),
    (14, 1, 4, (RX, RY, RZ), RING, 0, 12), (14, 1, 3, (RY, RZ), LADDER, 0, 11),
    (15, 1, 3, (RX, RY, RZ), RING, 0, 14), (14, 1, 2, (RY, RZ), LADDER, 0, 14), (13, 2, 2, (RY, RZ), RING, 1, 14),
    (16, 1, 3, (RY, RZ), RING, 0, 14),
]


@pytest.mark.parametrize("n,rows,L,rot,ent,reup,tile", CASES)
@pytest.mark.parametrize("inverse", [0, 1])
def test_plan_replay_matches_oracle(oracle, n, rows, L, rot, ent, reup, tile, inverse):
    g = np.random.Generator(np.random.PCG64(1000 + 13 * n + L + ent + 2 * reup + inverse))
    circ = qb.make_circuit(L, list(rot), ent, reup)
    P = qb.qsv_num_params(circ, n)
    ocirc = oracle.make_circuit(L, list(rot), ent, reup)
    assert P == oracle.num_params(ocirc, n)
    params = g.uniform(0, 2 * np.pi, P).astype(np.float32)
    feats = g.standard_normal((rows, n)).astype(np.float32) if reup else None
    x = g.standard_normal((rows, 1 << n)).astype(np.float32)
    ref, _ = oracle.amp_encode(x, n)
    start = ref.copy()
    oracle.apply_layers(ref, ocirc, params, feats, inverse=bool(inverse))
    text = qb.qsv_plan_describe(circ, n, rows, inverse, tile)
    out, n_gates, n_pass = replay(text, n, rows, L, rot, ent, reup, params.astype(np.float64),
                                  None if feats is None else feats.astype(np.float64), inverse, start)
    ent_gates = n if (ent == RING and n >= 2) else (n - 1 if ent == LADDER else 0)
    per_layer = (n if (reup + len(rot)) else 0) + ent_gates
    assert n_gates == L * per_layer                    # every gate exactly once
    assert np.allclose(out, ref, atol=1e-12)


DEFER = 0x100       # flag bit of qsv_plan_describe's tile argument: the plan with deferred CNOTs

DEFER_CASES = [
    # n, L, rot, tile
    (13, 3, (RY, RZ), 10), (14, 4, (RX, RY, RZ), 10), (15, 5, (RY, RZ), 11), (16, 4, (RX, RY, RZ), 12),
    (17, 6, (RY,), 12), (16, 3, (), 10), (18, 4, (RY, RZ), 13), (18, 3, (RX, RY, RZ), 14), (17, 5, (RZ, RX), 10),
]


@pytest.mark.parametrize("n,L,rot,tile", DEFER_CASES)
@pytest.mark.parametrize("inverse", [0, 1])
def test_plan_with_deferred_cnots_replays_to_the_oracle(oracle, n, L, rot, tile, inverse):
    """CNOTs whose target lies outside a pass's tile are carried by the pass's index map; replayed at
    the level of positions (register CNOTs under parities, the map applied at the store), the plan must
    still be the oracle's circuit, with fewer passes than the plan without deferral."""
    g = np.random.Generator(np.random.PCG64(9000 + 17 * n + L + inverse))
    circ = qb.make_circuit(L, list(rot), RING, 0)
    ocirc = oracle.make_circuit(L, list(rot), RING, 0)
    P = qb.qsv_num_params(circ, n)
    params = g.uniform(0, 2 * np.pi, P).astype(np.float32)
    x = g.standard_normal((1, 1 << n)).astype(np.float32)
    ref, _ = oracle.amp_encode(x, n)
    start = ref.copy()
    oracle.apply_layers(ref, ocirc, params, None, inverse=bool(inverse))
    text = qb.qsv_plan_describe(circ, n, 1, inverse, tile | DEFER)
    out, n_gates, n_pass = replay(text, n, 1, L, rot, RING, 0, params.astype(np.float64), None, inverse, start)
    assert n_gates == L * ((n if rot else 0) + n)
    assert np.allclose(out, ref, atol=1e-12)
    plain = qb.qsv_plan_describe(circ, n, 1, inverse, tile)
    assert " V" not in plain and " M" not in plain and " Q" not in plain
    assert n_pass <= sum(1 for ln in plain.split("\n") if ln.startswith("P "))
    if n - tile >= 3 and L >= 3:
        assert " V" in text and " M" in text       # the case is meant to exercise deferral


def test_plan_pass_counts_for_the_large_configs():
    """Pass counts decide the HBM traffic of the 20- and 26-qubit configs; pin their budget."""
    c3 = qb.make_circuit(20, [RY, RZ], RING)
    c4 = qb.make_circuit(30, [RX, RY, RZ], RING)
    for circ, n, B, layers in ((c3, 20, 32, 20), (c4, 26, 1, 30)):
        for inv in (0, 1):
            head, passes = parse_plan(qb.qsv_plan_describe(circ, n, B, inv, 0))
            assert len(passes) <= 2.8 * layers
            assert sum(h["gates"] for h, _ in passes) == layers * 2 * n


def test_bad_descriptors_are_rejected():
    assert qb.qsv_num_params(qb.make_circuit(1, [7], RING), 4) == -1
    assert qb.qsv_num_params(qb.make_circuit(-1, [RX], RING), 4) == -1
    assert qb.qsv_num_params(qb.make_circuit(1, [RX], 5), 4) == -1
    assert qb.qsv_num_params(qb.make_circuit(1, [RX], RING), 31) == -1
    assert qb.qsv_num_params(qb.make_circuit(3, [RX, RZ], LADDER, 1), 5) == 3 * 3 * 5
    assert qb.qsv_workspace_bytes(0, 1) == 0 and qb.qsv_workspace_bytes(4, 0) == 0
    with pytest.raises(ValueError):
        qb.qsv_plan_describe(qb.make_circuit(1, [RX], RING), 4, 1, 0, 9)


def _random_cases(count, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    rots = [(RX,), (RY,), (RZ,), (RY, RZ), (RZ, RX), (RX, RY, RZ), (RZ, RY, RX), ()]
    out = []
    for _ in range(count):
        n = int(g.integers(4, 17))
        rows = int(g.integers(1, 6)) if n <= 11 else 1
        L = int(g.integers(1, 5))
        rot = rots[int(g.integers(0, len(rots)))]
        ent = int(g.integers(0, 3))
        reup = int(g.integers(0, 2))
        if not rot and not reup and ent == NONE:
            ent = RING
        tile = int(g.choice([0, 10, 11, 12, 13, 14]))
        out.append((n, rows, L, rot, ent, reup, tile, int(g.integers(0, 2))))
    return out


@pytest.mark.parametrize("n,rows,L,rot,ent,reup,tile,inverse", _random_cases(60, 4242))
def test_plan_replay_random_circuits(oracle, n, rows, L, rot, ent, reup, tile, inverse):
    """Seeded sweep over qubit counts, batch sizes, rotation lists, entanglers, tile sizes and both
    directions: every plan, replayed operation by operation, must be the oracle's circuit."""
    g = np.random.Generator(np.random.PCG64(7000 + 31 * n + 7 * L + ent + 2 * reup + inverse + tile))
    circ = qb.make_circuit(L, list(rot), ent, reup)
    ocirc = oracle.make_circuit(L, list(rot), ent, reup)
    P = qb.qsv_num_params(circ, n)
    params = g.uniform(0, 2 * np.pi, P).astype(np.float32)
    feats = g.standard_normal((rows, n)).astype(np.float32) if reup else None
    x = g.standard_normal((rows, 1 << n)).astype(np.float32)
    ref, _ = oracle.amp_encode(x, n)
    start = ref.copy()
    oracle.apply_layers(ref, ocirc, params, feats, inverse=bool(inverse))
    text = qb.qsv_plan_describe(circ, n, rows, inverse, tile)
    out, n_gates, _ = replay(text, n, rows, L, rot, ent, reup, params.astype(np.float64),
                             None if feats is None else feats.astype(np.float64), inverse, start)
    ent_gates = n if (ent == RING and n >= 2) else (n - 1 if ent == LADDER else 0)
    per_layer = (n if (reup + len(rot)) else 0) + ent_gates
    assert n_gates == L * per_layer
    assert np.allclose(out, ref, atol=1e-12)


MIRROR = 0x200      # flag bit, with DEFER and inverse: the plan as the mirror of the circuit's own


@pytest.mark.parametrize("n,L,rot,tile", DEFER_CASES + [(19, 2, (RY, RZ), 0)])
def test_mirrored_plan_replays_to_the_oracle(oracle, n, L, rot, tile):
    """The inverse circuit's plan as the mirror of the circuit's plan: every pass with a map reads position p
    from the index that p maps to, applies its operations and writes positions as they are."""
    g = np.random.Generator(np.random.PCG64(9100 + 17 * n + L))
    circ = qb.make_circuit(L, list(rot), RING, 0)
    params = g.uniform(0, 2 * np.pi, qb.qsv_num_params(circ, n)).astype(np.float32)
    ref, _ = oracle.amp_encode(g.standard_normal((1, 1 << n)).astype(np.float32), n)
    st = ref.copy()
    oracle.apply_layers(ref, oracle.make_circuit(L, list(rot), RING, 0), params, None, inverse=True)
    batch = 8 if tile == 0 else 1
    forward = qb.qsv_plan_describe(circ, n, batch, 0, tile | DEFER).strip().split("\n")
    lines = qb.qsv_plan_describe(circ, n, batch, 1, tile | DEFER | MIRROR).strip().split("\n")
    assert len(lines) == len(forward)
    for line in lines[1:]:
        toks = line.split()
        maps = [t for t in toks if t[0] == "M"]
        if maps:
            imap = [int(x, 16) for x in maps[0][1:].split(",")]
            k = np.arange(1 << n)
            src = np.zeros(1 << n, dtype=np.int64)
            for j in range(n):
                src ^= np.where((k >> j) & 1, imap[j], 0)
            st = st[:, src]
        one = lines[0] + "\n" + " ".join(t for t in toks if t[0] != "M") + "\n"
        st, _, _ = replay(one, n, 1, L, rot, RING, 0, params.astype(np.float64), None, 1, st)
    assert np.allclose(st, ref, atol=1e-12)


@pytest.mark.parametrize("n", [18, 19, 20, 21, 22, 24, 26, 27, 28])
def test_default_tile_never_costs_a_pass(n):
    """The tile that a ring circuit gets by its number of qubits and layers takes no more passes than a tile of 2^12, and
    from 26 qubits on none more than 2^13 either."""
    def passes(L, batch, tile):
        circ = qb.make_circuit(L, [RY, RZ], 1, 0)
        return sum(ln.startswith("P ") for ln in qb.qsv_plan_describe(circ, n, batch, 0, tile | DEFER).split("\n"))

    for L in (1, 2, 3, 4, 5, 8, 9):
        for batch in (1, 8) if n < 24 else (1,):
            if batch << n <= 1 << 19:
                continue                             # tiles of 2^11 there, for the number of workgroups
            got, p12, p13 = passes(L, batch, 0), passes(L, 1, 12), passes(L, 1, 13)
            assert got <= p12, (L, batch)
            if n >= 26:
                assert got <= p13, (L, batch)


@pytest.mark.parametrize("ent,flag", [(RING, DEFER), (RING, 0), (LADDER, 0), (NONE, 0)])
def test_no_plan_has_fewer_passes_than_the_reverse_mode_sweep_expects(ent, flag):
    """The bound by which a circuit whose states cannot fit the workspace is not planned at all."""
    fewest = qb.load()["_ZN3qsv13fewest_passesERK11qsv_circuitii"]
    grows = 0
    for n in (10, 11, 13, 14, 16, 19, 20, 23):
        for tile in (10, 12, 13):
            for L in (1, 2, 3, 5, 8, 21):
                if n < tile:
                    continue
                circ = qb.make_circuit(L, [RY, RZ], ent)
                passes = sum(ln.startswith("P ") for ln in qb.qsv_plan_describe(circ, n, 1, 0, tile | flag).split("\n"))
                bound = fewest(ctypes.byref(circ), n, tile)
                assert 1 <= bound <= passes, (n, tile, L)
                grows = max(grows, bound)
    assert grows == {RING: 11, LADDER: 3, NONE: 1}[ent]
