"""The work users have this library do, as timed cases: batched fitness of given circuits (one
width or mixed widths, FP32 and FP64), circuit unitaries, and whole searches (QEQEA and GA
generations replayed from a HIP graph), each through the public entry points of
paper_1809_11134_amd.qe.

A case is a dict of plain values; `listed()` gives the standing ones, `draw(rng)` one more of the
same ranges.  `prepare` makes seeded inputs on the GPU, `run` is one pass, `work` the bytes and
operations a pass cannot do without, `exact` its outputs in 64 bits (plain torch)."""
import math

import numpy as np
import torch

# Descriptor kinds (bits 0-3 of a gate), target wire in bits 4-7, control in bits 8-11.
I_, NOT, CNOT, CV, CVDG, H, T = range(7)
RX, RY, RZ, ZZ = 7, 8, 9, 10

# The largest drawn batch costs no more than the largest listed one: 8192 circuits of 48 gates on
# six wires (circuit matrices times gates).
MAX_EVAL = 8192 * 48 * 4 ** 6


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest evaluation a user makes: one GA population of the paper's three-wire
        # problems; launch and call latency
        dict(name="eval_n3_b64_l10", kind="eval", n=3, lib="ncv", B=64, L=10, mode="eq11"),
        # an ordinary population of reversible circuits against one target
        dict(name="eval_n4_b4096_l30", kind="eval", n=4, lib="ncv", B=4096, L=30, mode="eq11"),
        # the largest uniform batch: six wires, circuits near a target of {H, T, CNOT, CV, CV+}
        dict(name="eval_n6_b8192_l48", kind="eval", n=6, lib="ht", B=8192, L=48, mode="eq11"),
        # uneven circuits of many problems in one call: widths 3..6, lengths 8..64, a target per
        # population of 64
        dict(name="eval_mixed_b16384", kind="mixed", B=16384),
        # FP64 check of candidate circuits kept outside a search
        dict(name="fp64_n5_b2048_l40", kind="fp64", n=5, lib="ht", B=2048, L=40),
        # the target unitaries of many problems, built on the GPU in FP64
        dict(name="unitary_n5_b1024_l16", kind="unitary", n=5, lib="perm", B=1024, L=16),
        # the throughput search: 1024 populations on five wires, generations and the FP64
        # re-check of each population's best
        dict(name="qeqea_n5_i1024_p64_l40", kind="qeqea", n=5, lib="ncv", I=1024, P=64, L=40,
             gens=50, mode="eq11", k=32, best=False),
        # one large population on four wires
        dict(name="qeqea_n4_p4096_l30", kind="qeqea", n=4, lib="ncv", I=1, P=4096, L=30,
             gens=50, mode="eq11", k=32, best=False),
        # a named-target convergence run between two reads of the best circuit (Toffoli-sized)
        dict(name="qeqea_n3_p256_l16", kind="qeqea", n=3, lib="ncv", I=1, P=256, L=16,
             gens=50, mode="phase", k=0, best=True),
        # the paper's own gate model, continuous angles
        dict(name="qeqea_ising_n4_p4096_l30", kind="qeqea", n=4, lib="ising", I=1, P=4096, L=30,
             gens=50, mode="eq11", k=32, best=False),
        # the classical baseline over populations of their own width and length
        dict(name="ga_mixed_i256_p64", kind="ga_mixed", I=256, P=64, gens=50),
        # the classical baseline with one large population (named-target runs)
        dict(name="ga_n4_p4096_l20", kind="ga", n=4, lib="ncv", I=1, P=4096, L=20, gens=50,
             mode="phase", best=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "mixed", "fp64", "unitary", "qeqea", "qeqea", "ga", "ga_mixed"])
    if kind == "eval":
        n, L = rng.randint(2, 6), _log_int(rng, 8, 64)
        lib = rng.choice(["ncv", "ht", "ising"])
        B = _log_int(rng, 64, max(64, min(16384, MAX_EVAL // (4 ** n * L))))
        # (the phase-insensitive fitness takes permutation targets)
        mode = "phase" if lib != "ht" and rng.random() < 0.3 else "eq11"
        return dict(kind=kind, n=n, lib=lib, B=B, L=L, mode=mode)
    if kind == "mixed":
        return dict(kind=kind, B=_log_int(rng, 256, 16384))
    if kind in ("fp64", "unitary"):
        n, L = rng.randint(2, 6), _log_int(rng, 8, 64)
        B = _log_int(rng, 32, max(32, min(4096, 4096 * 40 * 4 ** 5 // (4 ** n * L))))
        lib = rng.choice(["ht", "ncv", "ising"] if kind == "fp64" else ["perm", "ht"])
        return dict(kind=kind, n=n, lib=lib, B=B, L=L)
    if kind == "ga_mixed":
        return dict(kind=kind, I=_log_int(rng, 16, 256), P=rng.choice([32, 64, 100]), gens=20)
    mode = rng.choice(["eq11", "phase"])
    if kind == "ga":
        n, L, P = rng.randint(2, 6), rng.randint(8, 40), _log_int(rng, 64, 4096)
        I = _log_int(rng, 1, max(1, 16384 // P))
        return dict(kind=kind, n=n, lib="ncv", I=I, P=P, L=L, gens=20, mode=mode, best=I == 1)
    n, L, P = rng.randint(2, 6), rng.randint(10, 48), _log_int(rng, 64, 4096)
    I = _log_int(rng, 1, max(1, 32768 // P))
    lib = rng.choice(["ncv", "ncv", "ising"])
    return dict(kind=kind, n=n, lib=lib, I=I, P=P, L=L, gens=20, mode=mode,
                k=rng.choice([0, min(P, 32)]), best=I == 1)


# -------------------------------------------------------------------------- inputs
def _desc(kind, tgt=0, ctl=0):
    return kind | (tgt << 4) | (ctl << 8)


def _library(lib, n):
    pairs = [(c, t) for c in range(n) for t in range(n) if t != c]
    if lib == "perm":
        out = [_desc(NOT, w) for w in range(n)] + [_desc(CNOT, t, c) for c, t in pairs]
    else:
        out = ([_desc(I_)] + [_desc(NOT, w) for w in range(n)] if lib == "ncv" else
               [_desc(H, w) for w in range(n)] + [_desc(T, w) for w in range(n)])
        for c, t in pairs:
            out += [_desc(CNOT, t, c), _desc(CV, t, c), _desc(CVDG, t, c)]
    return np.array(out, np.int16)


def _random(rng, lib, n, shape):
    """Random gates, and their angles (None for the discrete libraries)."""
    if lib != "ising":
        tab = _library(lib, n)
        return tab[rng.integers(0, len(tab), size=shape)], None
    kind = rng.integers(RX, ZZ + 1 if n > 1 else ZZ, size=shape)
    a = rng.integers(0, n, size=shape)
    b = (a + rng.integers(1, n, size=shape)) % n if n > 1 else a
    g = kind | (a << 4) | (np.where(kind == ZZ, b, 0) << 8)
    ang = rng.integers(0, 1 << 32, size=shape, dtype=np.uint64).astype(np.uint32)
    return g.astype(np.int16), ang.view(np.int32)


def _planted(rng, lib, n, B, L):
    """A target's gate list of about 5/6 L gates, and B circuits of L: a quarter uniformly
    random, the others the target's list with 0..8 random substitutions."""
    tab = _library(lib, n)
    tg = tab[rng.integers(0, len(tab), size=max(1, 5 * L // 6))]
    g = tab[rng.integers(0, len(tab), size=(B, L))]
    near = np.arange(B) >= B // 4
    g[near] = np.concatenate([tg, np.zeros(L - len(tg), np.int16)])
    edits = rng.integers(0, 9, size=B)
    for e in range(8):
        rows = np.nonzero(near & (edits > e))[0]
        g[rows, rng.integers(0, L, size=len(rows))] = tab[rng.integers(0, len(tab), size=len(rows))]
    return tg, g


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _product(gates, angles, n, M):
    """U M in complex128 for circuits gates [B, L] (angles: u32 turn fractions in int32 storage,
    or None), M [B, 2^n, 2^n] or one matrix for all; gate 0 acts first, wire 0 is the highest bit
    of a row index."""
    dev, N = _dev(), 1 << n
    gates = torch.as_tensor(gates, device=dev).to(torch.int64)
    M = M.to(dev).expand(gates.shape[0], N, N).to(torch.complex128)
    r = torch.arange(N, device=dev)
    s = math.sqrt(0.5)
    one = np.eye(2, dtype=np.complex128)
    x = one[::-1]
    v = np.array([[1 + 1j, 1 - 1j], [1 - 1j, 1 + 1j]]) / 2
    tab = torch.tensor(np.array([one, x, x, v, v.conj(), [[s, s], [s, -s]], [[1, 0], [0, s + s * 1j]],
                                 one, one, one, one]), device=dev)
    ang = None if angles is None else torch.as_tensor(angles, device=dev).to(torch.int64) & 0xFFFFFFFF
    for l in range(gates.shape[1]):
        d = gates[:, l]
        kind, tp, cp = d & 15, n - 1 - ((d >> 4) & 15), n - 1 - ((d >> 8) & 15)
        bt, bc = (r >> tp[:, None]) & 1, (r >> cp[:, None].clamp(min=0)) & 1
        G = tab[kind].clone()
        if ang is not None:
            h = ang[:, l].to(torch.float64) * (math.pi / 2 ** 32)
            co, si = torch.cos(h).to(torch.complex128), torch.sin(h).to(torch.complex128)
            rot = [torch.stack([co, -1j * si, -1j * si, co], 1), torch.stack([co, -si, si, co], 1),
                   torch.stack([co - 1j * si, 0 * co, 0 * co, co + 1j * si], 1)]
            for k, m in zip((RX, RY, RZ), rot):
                G = torch.where((kind == k)[:, None, None], m.reshape(-1, 2, 2), G)
        b = torch.arange(len(d), device=dev)[:, None]
        A, C = G[b, bt, bt], G[b, bt, 1 - bt]
        on = ((kind != CNOT) & (kind != CV) & (kind != CVDG))[:, None] | (bc == 1)
        A, C = torch.where(on, A, torch.ones_like(A)), torch.where(on, C, torch.zeros_like(C))
        if ang is not None:
            ph = torch.where(bt == bc, (co - 1j * si)[:, None], (co + 1j * si)[:, None])
            A = torch.where((kind == ZZ)[:, None], ph, A)
        P = r ^ (1 << tp[:, None])
        M = A[:, :, None] * M + C[:, :, None] * M.gather(1, P[:, :, None].expand(-1, -1, N))
    return M


def _unitary(gates, n):
    return _product(gates, None, n, torch.eye(1 << n, dtype=torch.complex128)[None])


def _adjoint(U):
    return U.transpose(-1, -2).conj().contiguous()


def _perm_targets(rng, n, I, length):
    """I permutation targets, each a product of `length` random NOT/CNOT gates."""
    return _unitary(_random(rng, "perm", n, (I, length))[0], n)


def _eval_inputs(case, seed):
    rng = np.random.default_rng([seed, 1])
    n, B, L = case["n"], case["B"], case["L"]
    if case["lib"] == "ht":
        tg, gates = _planted(rng, "ht", n, B, L)
        return gates, None, _unitary(tg[None], n)
    gates, ang = _random(rng, case["lib"], n, (B, L))
    return gates, ang, _perm_targets(rng, n, 1, 12)


def _mixed_inputs(case, seed):
    """Populations of 64 circuits that share a width (3..6) and a target; every circuit has its
    own length (8..64)."""
    rng = np.random.default_rng([seed, 2])
    B = case["B"]
    pops = (B + 63) // 64
    widths, lens = rng.integers(3, 7, size=pops), rng.integers(8, 65, size=B)
    nq = np.repeat(widths, 64)[:B]
    goff = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gates = np.zeros(goff[-1], np.int16)
    pos_n = np.repeat(nq, lens)
    targets, toff = [None] * pops, np.concatenate([[0], np.cumsum(4 ** widths.astype(np.int64))])
    for n in range(3, 7):
        gates[pos_n == n] = _random(rng, "ht", n, int((pos_n == n).sum()))[0]
        which = np.nonzero(widths == n)[0]
        tg = _random(rng, "ht", n, (len(which), 40))[0]
        tg[np.arange(40)[None] >= rng.integers(8, 41, size=len(which))[:, None]] = 0
        for p, U in zip(which, _unitary(tg, n)):
            targets[p] = U.reshape(-1)
    return nq.astype(np.int8), goff, gates, np.repeat(toff[:-1], 64)[:B], torch.cat(targets)


# ------------------------------------------------------------------------- prepare
def prepare(case, seed):
    from paper_1809_11134_amd import qe
    dev, kind = _dev(), case["kind"]
    mode = qe.FIT_PHASE_INSENSITIVE if case.get("mode") == "phase" else qe.FIT_EQ11
    s = dict(case=case, mode=mode)
    if kind in ("eval", "fp64"):
        gates, ang, U = _eval_inputs(case, seed)
        s["gates"] = torch.from_numpy(gates).to(dev)
        s["angles"] = None if ang is None else torch.from_numpy(ang).to(dev)
        s["targets"] = U.to(torch.complex64 if kind == "eval" else torch.complex128)
    elif kind == "mixed":
        nq, goff, gates, toff, targets = _mixed_inputs(case, seed)
        s.update(nq=torch.from_numpy(nq).to(dev), goff=torch.from_numpy(goff).to(dev),
                 gates=torch.from_numpy(gates).to(dev), toff=torch.from_numpy(toff).to(dev),
                 targets=targets.to(torch.complex64))
        s["work"] = qe.eval_workspace(case["B"], dev)
    elif kind == "unitary":
        rng = np.random.default_rng([seed, 3])
        s["gates"] = torch.from_numpy(_random(rng, case["lib"], case["n"], (case["B"], case["L"]))[0]).to(dev)
    else:
        rng = np.random.default_rng([seed, 4])
        I, P, gens = case["I"], case["P"], case["gens"]
        if kind == "ga_mixed":
            # (the case's own widths and lengths; the seed draws targets and genomes)
            shape = np.random.default_rng([I, P])
            widths, lengths = shape.integers(3, 7, size=I), shape.integers(8, 65, size=I)
            targets = [None] * I
            for n in range(3, 7):
                which = np.nonzero(widths == n)[0]
                tg = _random(rng, "ht", n, (len(which), 24))[0]
                for i, U in zip(which, _unitary(tg, n)):
                    targets[i] = U.reshape(-1)
            ctx = qe.Context(0, qe.LIB_HT_NCV, qe.ALG_GA, 0, P, seed=seed, widths=widths.tolist(),
                             lengths=lengths.tolist())
            ctx.set_targets(torch.cat(targets))
        else:
            n = case["n"]
            lib = qe.LIB_ISING if case["lib"] == "ising" else qe.LIB_NCV
            alg = qe.ALG_GA if kind == "ga" else qe.ALG_QEQEA
            ctx = qe.Context(n, lib, alg, case["L"], P, I, seed=seed, fitness_mode=mode)
            ctx.set_targets(_perm_targets(rng, n, I, 12 if n < 5 else 16))
        s.update(ctx=ctx, gen=0, hist=torch.empty((gens, I, P), dtype=torch.float32, device=dev))
        ctx.graph_prepare(gens, s["hist"])
    return s


# ----------------------------------------------------------------------------- run
def run(s):
    from paper_1809_11134_amd import qe
    case, kind = s["case"], s["case"]["kind"]
    if kind == "eval":
        return qe.eval_fitness(s["gates"], s["targets"], n=case["n"], L=case["L"], target_stride=0,
                               fitness_mode=s["mode"], angles=s["angles"])[0]
    if kind == "mixed":
        return qe.eval_fitness(s["gates"], s["targets"], nq=s["nq"], goff=s["goff"], toff=s["toff"],
                               target_stride=None, workspace=s["work"])[0]
    if kind == "fp64":
        return qe.eval_fitness_fp64(s["gates"], s["targets"], n=case["n"], L=case["L"], target_stride=0,
                                    angles=s["angles"])[0]
    if kind == "unitary":
        return qe.build_unitary(s["gates"], case["n"], case["L"], precision=1)
    # a search: `gens` generations as one graph, the encoding (or genomes) they leave, and what
    # the program reads of them
    ctx, hist = s["ctx"], s["hist"]
    ctx.run_graph(s["gen"], case["gens"], hist)
    s["gen"] += case["gens"]
    out = {"f": hist}
    if case.get("k"):
        out["elite"], out["elite_f64"] = ctx.elite_recheck(None, hist[-1], case["k"])
    names = ("theta", "qutrit", "best_f") if kind == "qeqea" else ("genomes0", "genomes1")
    for name in names:
        out[name] = ctx.state(name)
    if case.get("best"):
        gates, f32, _ = ctx.get_best(0, with_fp64=False)
        out["best"], out["best_gates"] = f32, np.array(gates, np.int32)
    return out


# ---------------------------------------------------------------------------- work
def _gate_flops(lib, n):
    """Mean FP32 operations of a gate on a 2^n x 2^n complex matrix: 6 for each of the N^2 / 2
    entries a CV or CV+ changes, 4 for each entry H (N^2) or T (N^2 / 2) changes, 6 for each of
    the N^2 entries of a rotation or interaction, none for I, NOT and CNOT (they only move
    rows)."""
    NN = 4.0 ** n
    if lib == "ising":
        return 6 * NN
    if lib == "perm":
        return 0.0
    pairs = n * (n - 1)
    if lib == "sampled":                 # a region of Eq. 10 decodes to CV or CV+ half the time
        return 3 * NN * 0.5 * pairs / (n + pairs)
    total = (1 + n if lib == "ncv" else 2 * n) + 3 * pairs
    return (2 * pairs * 3 * NN + (0 if lib == "ncv" else n * (4 + 2) * NN)) / total


def work(case):
    kind = case["kind"]
    if kind in ("eval", "fp64"):
        n, B, L = case["n"], case["B"], case["L"]
        real = 4 if kind == "eval" else 8
        return {"bytes": B * L * (6 if case["lib"] == "ising" else 2) + 2 * real * 4 ** n + real * B,
                "flops": B * (L * _gate_flops(case["lib"], n) + 4 * 4 ** n)}
    if kind == "unitary":
        n, B, L = case["n"], case["B"], case["L"]
        return {"bytes": B * (2 * L + 16 * 4 ** n), "flops": B * L * _gate_flops(case["lib"], n)}
    if kind == "mixed":
        B = case["B"]
        return {"bytes": B * (2 * 36 + 1 + 4 + 8 + 4) + (B + 63) // 64 * 8 * sum(4 ** n for n in range(3, 7)) / 4,
                "flops": B * sum(36 * _gate_flops("ht", n) + 4 * 4 ** n for n in range(3, 7)) / 4}
    I, P, gens = case["I"], case["P"], case["gens"]
    if kind == "ga_mixed":
        nn = sum(4 ** n for n in range(3, 7)) / 4
        return {"bytes": gens * I * (P * (36 * 4 + 8) + 8 * nn) + I * P * 36 * 8,
                "flops": gens * I * P * sum(36 * _gate_flops("ht", n) + 4 * 4 ** n for n in range(3, 7)) / 4}
    n, L = case["n"], case["L"]
    NN = 4 ** n
    if kind == "ga":
        # each gene read and written once a generation, the target, the fitness
        return {"bytes": gens * I * (P * (4 * L + 8) + 8 * NN) + I * P * L * 8,
                "flops": gens * I * P * (L * _gate_flops("ncv", n) + 4 * NN)}
    # an entry's slot: its angle, best angle and best fitness read and half of it written, the
    # qutrit and its best copy of a rotation slot; a mutating individual's angles (or qutrits)
    # read and written; the descriptors, the fitness, the target; at the end the state read out
    ising = case["lib"] == "ising"
    R = n + n * (n - 1) // (2 if ising else 1)
    entry = 24 + 72 * n / R + 2
    mutation = 0.1 * (0.5 * R * L * 12 + 0.5 * n * L * 52)
    read = I * P * L * (R * 8 * 2 + n * 24 * 2)
    return {"bytes": gens * I * (P * (L * entry + 4 + mutation) + 8 * NN) + read,
            "flops": gens * I * P * (L * _gate_flops("ising" if ising else "sampled", n) + 4 * NN)}


# --------------------------------------------------------------------------- exact
def _fitness(M, mode):
    """Eq. 11 through the residual of M = U T^dagger, or the energy off the diagonal."""
    N = M.shape[-1]
    d = torch.diagonal(M, dim1=-2, dim2=-1)
    eye = torch.eye(N, dtype=torch.bool, device=M.device)
    off = (M.abs() ** 2).masked_fill(eye, 0).sum((-1, -2))
    if mode == "phase":
        r = off / N
    else:
        tr = d.sum(-1)
        ph = torch.where(tr.abs() > 0, tr / tr.abs().clamp(min=1e-300), torch.ones_like(tr))
        r = 0.5 * (off + ((d - ph[:, None]).abs() ** 2).sum(-1)) / N
    return 1 - torch.sqrt(r.clamp(0, 1))


def _chunked(fn, B, n):
    step = max(1, (1 << 24) // 4 ** n)
    return torch.cat([fn(slice(b, min(B, b + step))) for b in range(0, B, step)])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("eval", "fp64"):
        gates, ang, U = _eval_inputs(case, seed)
        # (the inputs of the FP32 call are rounded to 32 bits)
        U = _adjoint(U.to(torch.complex64).to(torch.complex128) if kind == "eval" else U)
        return _chunked(lambda c: _fitness(_product(gates[c], None if ang is None else ang[c], case["n"], U),
                                           case.get("mode", "eq11")), case["B"], case["n"])
    if kind == "unitary":
        rng = np.random.default_rng([seed, 3])
        return _unitary(_random(rng, case["lib"], case["n"], (case["B"], case["L"]))[0], case["n"])
    if kind == "mixed":
        nq, goff, gates, toff, targets = _mixed_inputs(case, seed)
        targets = targets.to(torch.complex64).to(torch.complex128)
        out = torch.zeros(case["B"], dtype=torch.float64, device=targets.device)
        for n in range(3, 7):
            which = np.nonzero(nq == n)[0]
            if not len(which):
                continue
            g = np.zeros((len(which), 64), np.int16)
            for j, b in enumerate(which):
                g[j, :goff[b + 1] - goff[b]] = gates[goff[b]:goff[b + 1]]
            at = torch.from_numpy(toff[which]).to(targets.device)
            sub = torch.arange(4 ** n, device=targets.device)

            def some(c):
                U = targets[at[c][:, None] + sub].reshape(-1, 1 << n, 1 << n)
                return _fitness(_product(g[c], None, n, _adjoint(U)), "eq11")
            out[torch.from_numpy(which).to(out.device)] = _chunked(some, len(which), n)
        return out
    return None                       # a search: its outputs follow its own random streams
