"""Performance cases of the encrypted iris-matching library.

Each case is one pass of what a program of this library has it do, through the entry points of the
package: a matching step (encode, encrypt, CCMM, decrypt, match) against a resident database in one
of the contraction forms, a batch of uneven requests through a reusable plan, the enrolment of a
database, FormatSwitch of transmitted queries, the fold of score ciphertexts.  Sizes are those of
the workloads in hfe_synth (tiny, mid, share) or generic ones of the same ranges.

listed() names the cases, draw(rng) gives another of the same ranges, prepare(case, seed) builds
what the program holds before the call, run(state) is the pass, work(case) counts the bytes and
operations the pass cannot do without, and exact(case, seed) gives the plain values in 64 bits.
"""
import math

import torch

import hfe_synth as S
import paper_2601_17561_amd as H

FORMS = {"digit": H.HFE_FORM_I8_MFMA, "rns": H.HFE_FORM_RNS_I8, "n2": H.HFE_FORM_P2_I8, "chain": H.HFE_FORM_P2_I8}
CHAIN_P_MODS = 3          # special moduli of the n^2 chain
TOP_WORK = 6.7e13         # operations of the largest listed case: the share step in the digit form
FOLD_COEFFS = (0.004105, -0.173510, -2.528271, 24.347349, 124.161550, -412.746212, 376.961251, 106.553952)


def listed():
    share = {"kind": "step", "log_n_db": 14, "log_n_q": 13, "level": 3, "d1": 14336, "d2": 12800, "eyes": 32,
             "shifts": 16, "row0": 0, "rows": 14336}
    return [
        # the smallest call: four unshifted codes against 256 of 1,024 bits (the tiny workload); launches count
        {"name": "step_tiny_digit", "kind": "step", "form": "digit", "log_n_db": 12, "log_n_q": 12, "level": 1,
         "d1": 256, "d2": 1024, "eyes": 4, "shifts": 1, "row0": 0, "rows": 256},
        # an ordinary small gallery with sizes that are ragged against every tile (the mid workload)
        {"name": "step_mid_rns", "kind": "step", "form": "rns", "log_n_db": 8, "log_n_q": 9, "level": 3, "d1": 700,
         "d2": 1280, "eyes": 17, "shifts": 16, "row0": 0, "rows": 700},
        # one GPU's share of the paper's gallery against 32 eyes in 16 shifts, in the forms a service picks from
        dict(share, name="step_share_digit", form="digit"),
        dict(share, name="step_share_rns", form="rns"),
        # the same over the paper's own modulus chain: seven query moduli n^2, three special ones
        dict(share, name="step_share_chain", form="chain", level=7),
        # one person at the gate: a single eye in 16 shifts against the share database
        dict(share, name="lookup_one_eye_rns", form="rns", eyes=1),
        # a few eyes against part of a mid-sized gallery, the n^2 form over the 36-bit primes, a query below the
        # database's level, odd sizes
        {"name": "step_ragged_n2", "kind": "step", "form": "n2", "log_n_db": 13, "log_n_q": 12, "level": 2, "d1": 9001,
         "d2": 9600, "eyes": 5, "shifts": 15, "row0": 513, "rows": 7777, "spare_primes": 1},
        # a serving step: twelve requests of 1..8 eyes at levels 1..3 on their own shards, a replayed plan
        {"name": "batch_plan_rns", "kind": "batch", "form": "rns", "log_n_db": 14, "log_n_q": 13, "level": 3,
         "d1": 14336, "d2": 12800, "items": 12, "max_eyes": 8, "shifts": 16, "min_rows": 2048, "mix": 5},
        # enrolment: the share's database encrypted for the digit form, then a first lookup against it
        {"name": "enrol_share_digit", "kind": "enrol", "form": "digit", "log_n_db": 14, "log_n_q": 13, "level": 3,
         "d1": 14336, "d2": 12800, "eyes": 1, "shifts": 1},
        # queries that arrive in the transmission ring 2^16 (512 columns), switched and matched on a small gallery
        {"name": "format_switch_512", "kind": "fs", "log_n_db": 10, "log_n_q": 13, "log_n_t": 16, "level": 3,
         "d1": 1024, "d2": 12800, "columns": 512},
        # the share's 1,024 score ciphertexts normalised and folded
        {"name": "fold_share", "kind": "fold", "log_n": 14, "k": 16, "rho": 512, "blocks": 2, "d2": 12800},
        # one eye's 16 score ciphertexts folded
        {"name": "fold_one_group", "kind": "fold", "log_n": 14, "k": 16, "rho": 16, "blocks": 1, "d2": 12800},
    ]


def _spread(rng, lo, hi):
    """An integer in lo..hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "batch", "enrol", "fs", "fold"))
    if kind == "fold":
        case = {"kind": "fold", "log_n": rng.randint(11, 14), "k": rng.choice((4, 8, 16)), "rho": _spread(rng, 6, 512),
                "blocks": rng.randint(1, 2), "d2": _spread(rng, 1000, 12800)}
    elif kind == "fs":
        lq = rng.randint(10, 13)
        case = {"kind": "fs", "log_n_db": rng.randint(8, 10), "log_n_q": lq, "log_n_t": rng.randint(lq, 16),
                "level": rng.randint(1, 3), "d1": _spread(rng, 100, 1024),
                "d2": _spread(rng, 1 << (lq - 1), min(12800, 2 << lq)), "columns": _spread(rng, 3, 512)}
    else:
        form = rng.choice(("digit", "rns", "rns", "n2") + (("chain",) if kind == "step" else ()))
        case = {"kind": kind, "form": form, "log_n_db": rng.randint(8, 14), "log_n_q": rng.randint(9, 13),
                "level": rng.randint(5, 7) if form == "chain" else rng.randint(1, 3), "d1": _spread(rng, 200, 14336),
                "d2": _spread(rng, 1000, 12800)}
        if kind == "step":
            case.update(eyes=_spread(rng, 1, 32), shifts=rng.choice((1, 3, 8, 15, 16, 16)))
            case["rows"] = rng.choice((case["d1"], rng.randint(case["d1"] // 2, case["d1"])))
            case["row0"] = rng.randint(0, case["d1"] - case["rows"])
        elif kind == "batch":
            case.update(items=rng.randint(2, 12), max_eyes=_spread(rng, 1, 8), shifts=rng.choice((8, 15, 16)),
                        min_rows=max(1, case["d1"] // 8), mix=rng.randint(0, 1 << 20))
        else:
            case.update(eyes=1, shifts=1)
    while work(case)["flops"] > TOP_WORK:
        for size in ("eyes", "max_eyes"):
            if size in case:
                case[size] = max(1, case[size] // 2)
    return case


# ---------------------------------------------------------------- inputs (from the seed alone)

def _rng(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + 7919 * stream) % (1 << 62))
    return g


def _bits(g, n, d2, p):
    return (torch.rand((n, d2), generator=g, device="cuda") < p).to(torch.uint8)


def _gallery(case, seed):
    g = _rng(seed, 1)
    return _bits(g, case["d1"], case["d2"], 0.5), _bits(g, case["d1"], case["d2"], 0.9)


def _eyes(case, seed, n, codes, masks, shifts, stream, row0=0, rows=None):
    """n query eyes; the first is a copy of a code of the rows matched, 10% of its bits flipped, rotated."""
    g = _rng(seed, stream)
    qc, qm = _bits(g, n, case["d2"], 0.5), _bits(g, n, case["d2"], 0.9)
    rows = case["d1"] if rows is None else rows
    row, back = row0 + (int(seed) * 31 + stream) % rows, -int(shifts[len(shifts) // 3])
    flip = _bits(g, 1, case["d2"], 0.1)[0]
    qc[0] = torch.roll(codes[row] ^ flip, back)
    qm[0] = torch.roll(masks[row], back)
    return qc, qm


def _keys(case, seed):
    if case.get("form") == "chain":
        return H.hfe_chain_keygen(H.hfe_chain_default_params(case["log_n_db"], case["log_n_q"], case["level"],
                                                             CHAIN_P_MODS, case["d2"], case["d1"]), seed + 1)
    spare = 1 if case["kind"] == "fs" else case.get("spare_primes", 0)
    return H.hfe_keygen(H.hfe_default_params(case["log_n_db"], case["log_n_q"], case["level"] + spare, case["d2"],
                                             case["d1"]), seed + 1)


def _shifts(case):
    return [int(s) for s in S.default_shifts(case["shifts"])]


def _mix(case):
    return S.batched_mix(case["mix"], case["items"], case["d1"], case["max_eyes"], case["level"], case["min_rows"])


def _scores(case, seed):
    """(ip, counts) of the fold: Binomial-like mask counts, scores of the non-matching law, one match per group."""
    n, slots, g = case["blocks"] * case["rho"], (1 << case["log_n"]) // 2, _rng(seed, 3)
    sd = math.sqrt(case["d2"] * 0.81 * 0.19)
    counts = torch.round(torch.randn((n, slots), generator=g, device="cuda") * sd + 0.81 * case["d2"])
    counts = counts.clamp(1, case["d2"])
    scores = (torch.randn((n, slots), generator=g, device="cuda") * 0.06 + 0.008).clamp(-0.233, 0.3)
    scores[:: case["k"], int(seed) % slots] = 0.45
    return torch.round(scores * counts).to(torch.int32), counts.to(torch.int32)


# ---------------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind, st = case["kind"], {"case": case, "seed": int(seed)}
    if kind == "fold":
        ip, counts = _scores(case, seed)
        st["keys"] = H.hfe_fold_keygen(case["log_n"], case["k"], case["rho"], seed + 1)
        st["ct"] = H.hfe_fold_encrypt(st["keys"], ip, seed + 2)
        st["counts"] = counts
        return st
    codes, masks = _gallery(case, seed)
    m_db = H.hfe_encode(codes, masks, [0])
    st["keys"] = _keys(case, seed)
    if kind == "fs":
        g = _rng(seed, 2)
        m_q = H.hfe_encode(_bits(g, case["columns"], case["d2"], 0.5), _bits(g, case["columns"], case["d2"], 0.9), [0])
        st["db"] = H.hfe_encrypt_db(st["keys"], m_db, seed + 3, H.HFE_FORM_RNS_I8)
        st["fk"] = H.hfe_fs_keygen(st["keys"], case["level"], case["log_n_t"], seed + 4)
        st["T"] = H.hfe_fs_encrypt(st["fk"], m_q, seed + 5)
        return st
    st["shifts"] = _shifts(case)
    if kind == "enrol":
        st["m_db"] = m_db
        qc, qm = _eyes(case, seed, 1, codes, masks, st["shifts"], 2)
        st["q"] = H.hfe_encrypt(st["keys"], H.hfe_encode(qc, qm, st["shifts"]), case["level"], seed + 4)
        return st
    st["db"] = H.hfe_encrypt_db(st["keys"], m_db, seed + 3, FORMS[case["form"]])
    if kind == "step":
        st["qc"], st["qm"] = _eyes(case, seed, case["eyes"], codes, masks, st["shifts"], 2, case["row0"], case["rows"])
        st["masks"] = masks[case["row0"]: case["row0"] + case["rows"]].contiguous()
        return st
    st["items"] = []
    for i, it in enumerate(_mix(case)):
        qc, qm = _eyes(case, seed, it.eyes, codes, masks, st["shifts"], 10 + i, it.row0, it.rows)
        q = H.hfe_encrypt(st["keys"], H.hfe_encode(qc, qm, st["shifts"]), it.level, seed + 10 + i)
        st["items"].append((q, it.row0, it.rows))
    st["plan"] = H.hfe_plan_create_for(st["db"], st["items"], FORMS[case["form"]])
    return st


def run(st):
    case, keys = st["case"], st["keys"]
    kind = case["kind"]
    if kind == "fold":
        return {"values": H.hfe_fold_decrypt(keys, H.hfe_fold(keys, st["ct"], st["counts"], case["rho"]))}
    if kind == "fs":
        q = H.hfe_format_switch(st["fk"], st["T"], case["columns"])
        v, ip = H.hfe_decrypt(keys, H.hfe_ccmm(st["db"], q, 0, case["d1"], H.HFE_FORM_RNS_I8))
        return {"v": v, "ip": ip}
    form = FORMS[case["form"]]
    if kind == "enrol":
        db = H.hfe_encrypt_db(keys, st["m_db"], st["seed"] + 3, form)
        v, ip = H.hfe_decrypt(keys, H.hfe_ccmm(db, st["q"], 0, case["d1"], form))
        return {"v": v, "ip": ip}
    if kind == "batch":
        H.hfe_plan_run(st["plan"], st["items"], use_graph=True)
        out = []
        for i in range(len(st["items"])):
            v, ip = H.hfe_decrypt(keys, H.hfe_plan_result(st["plan"], i))
            out.append({"v": v, "ip": ip})
        return out
    q = H.hfe_encrypt(keys, H.hfe_encode(st["qc"], st["qm"], st["shifts"]), case["level"], st["seed"] + 4)
    v, ip = H.hfe_decrypt(keys, H.hfe_ccmm(st["db"], q, case["row0"], case["rows"], form))
    decision, eye = H.hfe_match(ip, st["qm"], st["shifts"], st["masks"])
    return {"v": v, "ip": ip, "decision": decision, "eye": eye}


# ---------------------------------------------------------------- what a pass cannot do without

def _form_cost(form, K, level):
    """(stored bytes per database entry, int8 products per entry and query column) over the level's moduli and p."""
    if form == "chain":
        return 2 * (level + CHAIN_P_MODS), 3 * (level + CHAIN_P_MODS)
    nz = level + 1
    if form == "digit":
        return 5 * nz, 25 * nz
    bits = 72 + math.log2(K)  # the product of the small moduli holds four times the largest sum
    if form == "rns":
        n = math.ceil(bits / 7.9)
        return n * nz, n * nz
    n = math.ceil(bits / 15.75)
    return 2 * n * nz, 3 * n * nz


def _transform(log_n):
    return 6.0 * (1 << log_n) / 2 * log_n  # six fp64 operations per exact modular product


def work(case):
    kind = case["kind"]
    if kind == "fold":
        n, N, slots = case["blocks"] * case["rho"], 1 << case["log_n"], (1 << case["log_n"]) // 2
        folded = case["blocks"] * -(-case["rho"] // case["k"])
        # five relinearised products, four constant terms, the normalisation and a rotation: 148 transforms
        return {"bytes": n * (10 * N * 8 + slots * 4) + folded * slots * 8, "flops": 148 * n * _transform(case["log_n"])}
    N_db, K = 1 << case["log_n_db"], case["d2"] + (1 << case["log_n_q"])
    if kind == "batch":
        nbytes = flops = 0
        per, products = _form_cost(case["form"], K, case["level"])
        per, products = per / (case["level"] + 1), products / (case["level"] + 1)
        for it in _mix(case):
            cols = it.eyes * case["shifts"]
            flops += 2 * products * (it.level + 1) * (N_db + it.rows) * K * cols
            nbytes += cols * (it.rows * 12 + 8 * K * it.level)
        nbytes += (N_db + case["d1"]) * K * per * (max(it.level for it in _mix(case)) + 1)
        return {"bytes": nbytes, "flops": flops}
    if kind == "fs":
        cols, k, nz = case["columns"], -(-case["d2"] // (1 << case["log_n_q"])), case["level"] + 1
        per, products = _form_cost("rns", K, case["level"])
        rho = 1 << (case["log_n_t"] - case["log_n_q"])
        ring = cols * k * (nz + 1) * (nz * rho + 2) * _transform(case["log_n_q"])
        conv = cols * (nz + 1) * (nz * k + k + 1) * _transform(case["log_n_q"])
        return {"bytes": cols * k * nz * 2 * (8 << case["log_n_t"]) + (N_db + case["d1"]) * K * per
                + cols * case["d1"] * 12,
                "flops": ring + conv + 2.0 * products * (N_db + case["d1"]) * K * cols}
    cols = case["eyes"] * case["shifts"]
    per, products = _form_cost(case["form"], K, case["level"])
    if kind == "enrol":
        layers = 1 + -(-case["d1"] // N_db)
        ntt = K * (case["level"] + 1) * layers * _transform(case["log_n_db"])
        return {"bytes": case["d1"] * case["d2"] + (N_db + case["d1"]) * K * per + cols * case["d1"] * 12,
                "flops": ntt + 2.0 * products * (N_db + case["d1"]) * K * cols}
    rows = N_db + case["rows"]
    return {"bytes": rows * K * per + 2 * case["eyes"] * case["d2"] + case["rows"] * (case["d2"] + cols * 13),
            "flops": 2.0 * products * rows * K * cols}


# ---------------------------------------------------------------- plain values in 64 bits

def _ternary(codes, masks):
    c, m = codes.double(), masks.double()
    return m - 2 * c * m


def _rolled(x, shifts):
    return torch.stack([torch.roll(x, s, 1) for s in shifts], 1).reshape(-1, x.shape[1])


def exact(case, seed):
    kind = case["kind"]
    if kind == "fold":
        ip, counts = _scores(case, seed)
        x = ip.double() / counts.double()
        f = torch.zeros_like(x)
        for c in reversed(FOLD_COEFFS):
            f = f * x + c
        out, k, rho = [], case["k"], case["rho"]
        for b in range(case["blocks"]):
            for r in range(-(-rho // k)):
                out.append(sum(torch.roll(f[b * rho + r * k + i], r * k + i) for i in range(min(k, rho - r * k))))
        return {"values": torch.stack(out)}
    codes, masks = _gallery(case, seed)
    m_db = _ternary(codes, masks)
    if kind == "fs":
        g = _rng(seed, 2)
        ip = _ternary(_bits(g, case["columns"], case["d2"], 0.5), _bits(g, case["columns"], case["d2"], 0.9)) @ m_db.T
        return {"v": ip, "ip": ip.to(torch.int32)}
    shifts = _shifts(case)
    if kind == "batch":
        out = []
        for i, it in enumerate(_mix(case)):
            qc, qm = _eyes(case, seed, it.eyes, codes, masks, shifts, 10 + i, it.row0, it.rows)
            ip = _rolled(_ternary(qc, qm), shifts) @ m_db[it.row0: it.row0 + it.rows].T
            out.append({"v": ip, "ip": ip.to(torch.int32)})
        return out
    if kind == "enrol":
        qc, qm = _eyes(case, seed, 1, codes, masks, shifts, 2)
        ip = _rolled(_ternary(qc, qm), shifts) @ m_db.T
        return {"v": ip, "ip": ip.to(torch.int32)}
    lo, hi = case["row0"], case["row0"] + case["rows"]
    qc, qm = _eyes(case, seed, case["eyes"], codes, masks, shifts, 2, lo, case["rows"])
    ip = _rolled(_ternary(qc, qm), shifts) @ m_db[lo:hi].T
    overlap = _rolled(qm.double(), shifts) @ masks[lo:hi].double().T
    decision = ip * 8 > 2 * overlap
    return {"v": ip, "ip": ip.to(torch.int32), "decision": decision.to(torch.uint8),
            "eye": decision.reshape(case["eyes"], -1).any(1).to(torch.uint8)}
