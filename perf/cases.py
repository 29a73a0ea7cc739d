"""Performance cases of the library: what a program that evaluates CKKS circuits
on the GPU calls, from a transform of a few 4096-point limbs to a full-slot
bootstrap at N = 2^16, through the Python binding's public entry points.

A case names an operation, a parameter set of inputs.py and the sizes of the
call (level, limbs, rotations, items).  `listed` holds the fixed cases, `draw`
gives more of the same ranges, `prepare` builds a case's inputs on the GPU from
a seed, `run` makes the call, `work` says what it cannot do without.  Every
output is a residue, an exact whole number, so there is no floating-point
reference here.

Contexts (twiddles and conversion constants of a parameter set) and the
bootstrap's plaintext plan hold no input: a program makes them once, and they
are kept here for the same reason.  Keys, ciphertexts, plaintexts, outputs,
workspaces and the batch and bootstrap handles belong to a prepared state.
"""
from functools import lru_cache

import torch

from paper_2507_04775_amd import bootplan, ckks, inputs

# Level ranges per parameter set and the word size of the set's path.
SETS_64 = ("small", "small-nv", "boot-small", "large", "large-nv", "large-fp")
SETS_32 = ("w32-small", "w32-large")


@lru_cache(maxsize=None)
def param_set(name):
    return inputs.params32(name) if name in SETS_32 else inputs.params(name)


@lru_cache(maxsize=None)
def context(name):
    ps = param_set(name)
    kind = ckks.Context32 if name in SETS_32 else ckks.Context
    return kind(ps.logn, ps.q, ps.p, ps.dnum)


@lru_cache(maxsize=None)
def _boot(name, sparse, hoist, groups):
    """The package's schedule: the sine of the sparse or of the uniform secret,
    ModDown inside or outside the giant-step loops, the butterfly stages merged
    into two or three groups as even as possible."""
    ps = param_set(name)
    cfg = bootplan.default_config(ps.logn, 2.0 ** ps.log_scale, sparse=sparse)
    cfg.hoist_moddown = hoist
    stages = ps.logn - 1
    parts = [stages // groups + (1 if i < stages % groups else 0) for i in range(groups)]
    cfg.cts_radix_logs, cfg.stc_radix_logs = parts, parts[::-1]
    return cfg, bootplan.plan(ps.q, cfg)


def boot_config(case):
    return _boot(case["set"], case["sparse"], case["hoist"], case["groups"])


# ------------------------------------------------------------------- cases


def listed():
    return [
        # the smallest call there is: one plaintext's limbs into evaluation form in the N = 2^12 ring
        {"name": "ntt-2^12-4", "op": "ntt", "set": "small", "limbs": 4, "limb0": 0, "inverse": False},
        # every prime of the N = 2^16 set at once: an encoded plaintext, a fresh key row
        {"name": "ntt-2^16-35", "op": "ntt", "set": "large", "limbs": 35, "limb0": 0, "inverse": False},
        # back to coefficients in the middle of a circuit (decryption, re-encoding), an odd number of limbs
        {"name": "intt-2^16-13", "op": "ntt", "set": "large", "limbs": 13, "limb0": 0, "inverse": True},
        # a shallow circuit on small rings: the product is all launches and latency
        {"name": "hmult-2^12-l3", "op": "hmult", "set": "small", "level": 3},
        # the product of two fresh ciphertexts, the largest relinearisation
        {"name": "hmult-2^16-l30", "op": "hmult", "set": "large", "level": 30},
        # a rotation half way down a circuit: the last digit is partial
        {"name": "rotate-2^16-l17", "op": "rotate", "set": "large", "level": 17, "rot": 77},
        # the baby steps of a matrix-vector product: several rotations of one ciphertext, ten special primes
        {"name": "hoisted-2^16-l23x5", "op": "hoisted", "set": "large-nv", "level": 23, "n_rot": 5},
        # a * plaintext + b, rescaled: the linear layers' other half, no key
        {"name": "ptmuladd-2^16-l12", "op": "ptmuladd", "set": "large", "level": 12},
        # independent ciphertexts of mixed levels in one batch, products and eightfold rotations
        {"name": "batch-2^16x32", "op": "batch", "set": "large", "items": 32, "plan": 1},
        # a full-slot bootstrap, the package's default schedule
        {"name": "bootstrap-2^16", "op": "bootstrap", "set": "large-nv", "sparse": True, "hoist": True,
         "groups": 3},
        # the 32-bit word path: a fresh product, and a rotation with a partial last digit
        {"name": "hmult32-2^16-l51", "op": "hmult32", "set": "w32-large", "level": 51},
        {"name": "rotate32-2^16-l24", "op": "rotate32", "set": "w32-large", "level": 24, "rot": 513},
    ]


def _log_int(rng, lo, hi):
    """A whole number in [lo, hi], uniform in its logarithm."""
    return min(hi, int(lo * ((hi + 1) / lo) ** rng.random()))


def draw(rng):
    op = rng.choice(("ntt", "ntt", "hmult", "hmult", "rotate", "rotate", "keyswitch", "hoisted", "ptmuladd", "rescale",
                     "batch", "bootstrap", "hmult32", "rotate32", "rescale32", "ntt32"))
    c = {"op": op}
    if op.endswith("32"):
        c["set"] = rng.choice(("w32-small", "w32-large", "w32-large"))
    elif op == "bootstrap":
        c["set"] = "boot-small"
    elif op == "batch":
        c["set"] = rng.choice(("large", "large", "boot-small"))
    else:
        c["set"] = rng.choice(("small", "small-nv", "boot-small", "large", "large", "large", "large-nv", "large-fp"))
    ps = param_set(c["set"])
    if op in ("ntt", "ntt32"):
        n = ps.L + 1 + ps.K
        c["limbs"] = _log_int(rng, 1, n)
        c["limb0"] = rng.randrange(n - c["limbs"] + 1)
        c["inverse"] = rng.random() < 0.5
    elif op == "batch":
        c["items"] = _log_int(rng, 2, 32)
        c["plan"] = rng.randrange(1000)
    elif op == "bootstrap":
        c["sparse"], c["hoist"] = rng.random() < 0.6, rng.random() < 0.6
        c["groups"] = rng.choice((2, 3))
    else:
        low = 1 if op in ("ptmuladd", "rescale", "rescale32") else 0
        c["level"] = _log_int(rng, low + 1, ps.L + 1) - 1
        if op in ("rotate", "rotate32"):
            c["rot"] = rng.randrange(1, ps.N // 2)
        if op == "hoisted":
            c["n_rot"] = rng.randint(2, 8)
    return c


# ------------------------------------------------------------------ inputs


class _Draw:
    """Uniform residues on the device, every tensor from a seed of its own."""

    def __init__(self, seed):
        self.seed = (int(seed) & 0xFFFFFFFF) * 100003 + 17

    def rows(self, mods, N):
        self.seed += 1
        return inputs.device_residues(self.seed, mods, N)

    def poly(self, ps, level):
        return self.rows(ps.q[: level + 1], ps.N)

    def ct(self, ps, level):
        return ckks.Ciphertext(self.poly(ps, level), self.poly(ps, level), level, 2.0 ** ps.log_scale)

    def key_data(self, ps):
        mods = list(ps.q) + list(ps.p)
        return self.rows(mods * (2 * ps.dnum), ps.N).reshape(ps.dnum, 2, len(mods), ps.N)

    def words(self, t):
        """The same residues as 32-bit words (primes below 2^30)."""
        return t.view(torch.int64).to(torch.int32).contiguous()


def _galois(ps, k):
    return pow(5, k, 2 * ps.N)


def _batch_items(case):
    """The bench's mixed batch: half products, half hoisted eightfold rotations, levels 4 .. L."""
    ps = param_set(case["set"])
    return inputs.batch_plan(case["plan"], case["items"], ps.logn, ps.L)


def prepare(case, seed):
    op, ps, ctx, r = case["op"], param_set(case["set"]), context(case["set"]), _Draw(seed)
    s = {"op": op, "ctx": ctx, "level": case.get("level")}
    lv = case.get("level")
    if op == "ntt":
        mods = (list(ps.q) + list(ps.p))[case["limb0"]: case["limb0"] + case["limbs"]]
        s.update(poly=r.rows(mods, ps.N), limb0=case["limb0"], inverse=case["inverse"])
    elif op == "hmult":
        s.update(a=r.ct(ps, lv), b=r.ct(ps, lv), key=ctx.key(r.key_data(ps), 0), out=ctx.empty_ct(lv))
    elif op == "rotate":
        s.update(a=r.ct(ps, lv), rot=case["rot"], key=ctx.key(r.key_data(ps), _galois(ps, case["rot"])),
                 out=ctx.empty_ct(lv))
    elif op == "keyswitch":
        s.update(d=r.poly(ps, lv), key=ctx.key(r.key_data(ps), 0), out=ctx.empty_ct(lv))
    elif op == "hoisted":
        ks = inputs.batch_rotation_set(ps.logn)[: case["n_rot"]]
        s.update(a=r.ct(ps, lv), ks=ks, keys=[ctx.key(r.key_data(ps), _galois(ps, k)) for k in ks],
                 outs=[ctx.empty_ct(lv) for _ in ks])
    elif op == "rescale":
        s.update(a=r.ct(ps, lv), out=ctx.empty_ct(lv - 1))
    elif op == "ptmuladd":
        s.update(a=r.ct(ps, lv), b=r.ct(ps, lv), pt=r.poly(ps, lv), scale=2.0 ** ps.log_scale,
                 prod=ctx.empty_ct(lv), out=ctx.empty_ct(lv - 1))
    elif op == "batch":
        s.update(_prepare_batch(case, ps, ctx, r))
    elif op == "bootstrap":
        s.update(_prepare_boot(case, ps, ctx, r))
    elif op == "ntt32":
        mods = (list(ps.q) + list(ps.p))[case["limb0"]: case["limb0"] + case["limbs"]]
        s.update(poly=r.words(r.rows(mods, ps.N)), limb0=case["limb0"], inverse=case["inverse"])
    else:
        a = [r.words(r.poly(ps, lv)) for _ in range(4 if op == "hmult32" else 2)]
        kind = {"hmult32": ckks.OP_HMULT, "rotate32": ckks.OP_ROTATE, "rescale32": ckks.OP_RESCALE}[op]
        n = lv if op == "rescale32" else lv + 1
        s.update(a=a, out=[ctx.empty(n), ctx.empty(n)], ws=ctx.workspace(kind, lv))
        if op != "rescale32":
            s["key"] = r.words(r.key_data(ps))
        if op == "rotate32":
            s["galois"] = _galois(ps, case["rot"])
    return s


def _prepare_batch(case, ps, ctx, r):
    rlk, keys = ctx.key(r.key_data(ps), 0), {}
    batch, keep = ckks.Batch(ctx), []
    items = _batch_items(case)
    # the outputs are rows of one buffer, as a program that hands the batch's results on would keep them
    rows = sum(2 * (lv + 1) * (len(ks) if ks else 1) for _, lv, ks in items)
    buf, at = torch.empty((rows, ps.N), dtype=torch.uint64, device="cuda"), 0

    def out_ct(lv):
        nonlocal at
        n = lv + 1
        ct = ckks.Ciphertext(buf[at: at + n], buf[at + n: at + 2 * n], lv)
        at += 2 * n
        return ct

    for kind, lv, ks in items:
        a = r.ct(ps, lv)
        if kind == "hmult":
            b = r.ct(ps, lv)
            batch.hmult(a, b, rlk, out_ct(lv))
            keep += [a, b]
        else:
            for k in ks:
                if k not in keys:
                    keys[k] = ctx.key(r.key_data(ps), _galois(ps, k))
            batch.hoisted(a, ks, [keys[k] for k in ks], [out_ct(lv) for _ in ks])
            keep.append(a)
    return {"batch": batch.build(), "outputs": buf, "keep": keep, "rlk": rlk, "keys": keys}


def _prepare_boot(case, ps, ctx, r):
    cfg, pl = boot_config(case)
    relin, conj = ctx.key(r.key_data(ps), 0), ctx.key(r.key_data(ps), 2 * ps.N - 1)
    rot = {k: ctx.key(r.key_data(ps), _galois(ps, k)) for k in pl.rotations}
    sparse = (ctx.key(r.key_data(ps), 0), ctx.key(r.key_data(ps), 0)) if case["sparse"] else None
    boot = ckks.Boot(ctx, cfg.cts_radix_logs, cfg.stc_radix_logs, pl.cts, pl.stc, pl.cheb, cfg.double_angles,
                     cfg.top_scale, relin, conj, rot, cheb_baby=cfg.cheb_baby, sparse=sparse,
                     hoist_moddown=cfg.hoist_moddown, input_gain=cfg.input_gain)
    a = r.ct(ps, 0)
    return {"boot": boot, "a": a, "out": ctx.empty_ct(boot.output_level)}


# --------------------------------------------------------------------- run


def _whole(*polys):
    """The residues as they lie in memory (64-bit words seen as signed integers)."""
    return [p.view(torch.int64) if p.dtype == torch.uint64 else p for p in polys]


def run(s):
    op, ctx = s["op"], s["ctx"]
    if op == "ntt":  # in place, as the library's transforms are
        (ctx.ckks_intt if s["inverse"] else ctx.ckks_ntt)(s["poly"], s["limb0"])
        return _whole(s["poly"])
    if op == "ntt32":
        (ctx.intt if s["inverse"] else ctx.ntt)(s["poly"], s["limb0"])
        return _whole(s["poly"])
    if op == "hmult":
        ctx.ckks_hmult_relin(s["a"], s["b"], s["key"], s["out"])
    elif op == "rotate":
        ctx.ckks_hrotate(s["a"], s["rot"], s["key"], s["out"])
    elif op == "keyswitch":
        ctx.ckks_keyswitch(s["d"], s["level"], s["key"], s["out"].c0, s["out"].c1)
    elif op == "rescale":
        ctx.ckks_rescale(s["a"], s["out"])
    elif op == "ptmuladd":
        ctx.ckks_ptmult(s["a"], s["pt"], s["scale"], s["prod"])
        ctx.ckks_hadd(s["prod"], s["b"], s["prod"])
        ctx.ckks_rescale(s["prod"], s["out"])
    elif op == "hoisted":
        ctx.ckks_hrotate_hoisted(s["a"], s["ks"], s["keys"], s["outs"])
        return [_whole(o.c0, o.c1) for o in s["outs"]]
    elif op == "batch":
        s["batch"].run()
        return _whole(s["outputs"])
    elif op == "bootstrap":
        s["boot"].ckks_bootstrap(s["a"], s["out"])
    elif op == "hmult32":
        ctx.hmult_relin(*s["a"], s["level"], s["key"], *s["out"], ws=s["ws"])
        return _whole(*s["out"])
    elif op == "rotate32":
        ctx.apply_galois(*s["a"], s["level"], s["galois"], s["key"], *s["out"], ws=s["ws"])
        return _whole(*s["out"])
    elif op == "rescale32":
        ctx.rescale(*s["a"], s["level"], *s["out"], ws=s["ws"])
        return _whole(*s["out"])
    return _whole(s["out"].c0, s["out"].c1)


# -------------------------------------------------------------------- work
# Bytes: every input and output once.  Operations: a butterfly is a modular
# product, a sum and a difference (3); a term of a sum of products is 2.


def _transforms(ps, limbs):
    return 3 * limbs * (ps.N // 2) * ps.logn


def _modup(ps, level):
    n, rows = level + 1, level + 1 + ps.K
    terms = 0
    for lo in range(0, n, ps.alpha):
        ns = min(ps.alpha, n - lo)
        terms += ns * (rows - ns)
    return _transforms(ps, ps.beta(level) * rows) + 2 * terms * ps.N


def _ip_moddown(ps, level):
    n, rows = level + 1, level + 1 + ps.K
    return 4 * ps.beta(level) * rows * ps.N + _transforms(ps, 2 * ps.K + 2 * n) + 2 * 2 * ps.K * n * ps.N


def _key_words(ps, level):
    return 2 * ps.beta(level) * (level + 1 + ps.K) * ps.N


def _switches(ps, level, count=1):
    return count * (_modup(ps, level) + _ip_moddown(ps, level))


def work(case):
    op, ps = case["op"], param_set(case["set"])
    word = 4 if case["set"] in SETS_32 else 8
    lv = case.get("level") or 0
    n, N = lv + 1, ps.N
    if op in ("ntt", "ntt32"):
        words, ops = 2 * case["limbs"] * N, _transforms(ps, case["limbs"])
    elif op in ("hmult", "hmult32"):
        words, ops = 6 * n * N + _key_words(ps, lv), _switches(ps, lv) + 7 * n * N
    elif op in ("rotate", "rotate32"):
        words, ops = 4 * n * N + _key_words(ps, lv), _switches(ps, lv) + n * N
    elif op == "keyswitch":
        words, ops = 3 * n * N + _key_words(ps, lv), _switches(ps, lv)
    elif op == "hoisted":
        r = case["n_rot"]
        words, ops = (2 + 2 * r) * n * N + r * _key_words(ps, lv), _modup(ps, lv) + r * (_ip_moddown(ps, lv) + n * N)
    elif op in ("rescale", "rescale32"):
        words, ops = (2 * n + 2 * lv) * N, _transforms(ps, 2 + 2 * lv) + 4 * lv * N
    elif op == "ptmuladd":
        words, ops = (5 * n + 2 * lv) * N, _transforms(ps, 2 + 2 * lv) + 4 * lv * N + 4 * n * N
    elif op == "batch":
        words, ops, key_level = 0, 0, {}
        for kind, level, ks in _batch_items(case):
            m = level + 1
            if kind == "hmult":
                words, ops = words + 6 * m * N, ops + _switches(ps, level) + 7 * m * N
            else:
                words += (2 + 2 * len(ks)) * m * N
                ops += _modup(ps, level) + len(ks) * (_ip_moddown(ps, level) + m * N)
            for k in ks or (0,):
                key_level[k] = max(key_level.get(k, 0), level)
        words += sum(_key_words(ps, level) for level in key_level.values())
    else:
        words, ops = _boot_work(case, ps)
    return {"bytes": float(words * word), "flops": float(ops)}


def _boot_work(case, ps):
    """CoeffToSlot, EvalMod and SlotToCoeff at the levels they run at: every
    plaintext diagonal and every key's rows once; baby rotations share a ModUp."""
    cfg, _ = boot_config(case)
    words, ops, N = 0, 0, ps.N

    def group(level, radix, whole):
        R = 1 << radix
        count = R if whole else 2 * R - 1
        baby = 1
        while baby * baby < count:
            baby *= 2
        giants = -(-count // baby)
        w = count * (level + 1) * N + (baby + giants - 2) * _key_words(ps, level)
        o = _modup(ps, level) + (baby - 1) * _ip_moddown(ps, level) + _switches(ps, level, giants - 1)
        return w, o + 4 * count * (level + 1) * N

    level = ps.L
    for i, radix in enumerate(cfg.cts_radix_logs):
        w, o = group(level, radix, i == 0)
        words, ops, level = words + w, ops + o, level - (2 if i == 0 else 1)
    words, ops = words + _key_words(ps, level), ops + _switches(ps, level)  # the conjugation
    depth = bootplan.cheb_depth(cfg.cheb_degree, cfg.baby)
    products = 2 * (cfg.baby - 2 + 2 * (cfg.cheb_degree + 1) // cfg.baby)  # both halves
    words += _key_words(ps, level)
    for i in range(depth):
        ops += _switches(ps, level - i, products / depth)
    level -= depth
    for i in range(cfg.double_angles):
        ops += _switches(ps, level, 2)
        level -= 1
    for i, radix in enumerate(cfg.stc_radix_logs):
        w, o = group(level, radix, i == len(cfg.stc_radix_logs) - 1)
        words, ops, level = words + w, ops + o, level - 1
    return words + 2 * N + 2 * (level + 1) * N, ops
