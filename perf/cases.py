"""The work that a user of this package has it do, as timing cases over its public entry points.

A garbled inference has an offline side (Gb: draw the labels, garble every layer; ship the tables) and an online side
(En, Ev, De), so most cases come as a pair.  Networks are the shapes of the benchmark configurations and of the paper's
models (the table of model architectures), with random weights: run time does not depend on them.

  kind "net"     GarbledNetwork, all tables resident.  do = "garble"  Gb of the whole network
                                                       do = "infer"   En + Ev + De on tables garbled before
                                                       do = "ship"    Gb, then the packed storage format of tables and output labels
                                                       do = "receive" the packed tables back to the working format, then En + Ev + De
  kind "stream"  StreamedNetwork: networks whose tables do not fit at once, layer by layer, Gb + En + Ev + De
  kind "linear"  one dense or convolution layer on label tensors (the same arithmetic for garbler and evaluator)
  kind "proj"    ProjectionBatch: independent gates Z_p -> Z_q with mixed moduli.  do = "garble" or "eval"

rule: label lengths by "ceil" (at least 128 bits a label, the default) or "floor" (a label packs into 128 bits; the packed
formats need it).  digits: "exact" sign or the "reduced" accuracy set.
"""
import numpy as np
import torch

from paper_2302_06361_amd import CONV2D, DENSE, LAMBDA_CEIL, LAMBDA_FLOOR, Context, GarbledNetwork, Labels, Layer, ProjectionBatch, StreamedNetwork

PRIMES = [2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37]
# mixed-radix digits of the sign gadget by number of primes: exact sign
DIGITS = {7: (10,) + (13,) * 5, 8: (26,) + (12,) * 6, 9: (22,) + (10,) * 8, 12: (46,) + (17,) * 10}
REDUCED = {8: (26, 12, 12)}

# (out channels, filter, stride, pad) convolutions, "d" dense, "R" ReLU and rescaling, "P" 2x2 sum pooling
CONVNETS = {
    # the LeNet-5 shape of the benchmark's main configuration
    "lenet": dict(hw=28, c=1, k=8, repeat=6, layers=[(6, 5, 1, 2), "R", "P", (16, 5, 1, 0), "R", "P", ("d", 120), "R", ("d", 84), "R", ("d", 10)]),
    # the paper's models
    "A": dict(hw=28, c=1, k=8, repeat=0, layers=[("d", 128), "R", ("d", 128), "R", ("d", 10)]),
    "B": dict(hw=28, c=1, k=9, repeat=0, layers=[(5, 5, 1, 0), "R", (5, 3, 3, 0), "R", (10, 3, 1, 0), "R", (10, 3, 3, 0), "R", ("d", 100), "R", ("d", 10)]),
    "C": dict(hw=28, c=1, k=9, repeat=0, layers=[(5, 4, 2, 0), "R", ("d", 100), "R", ("d", 10)]),
    "D": dict(hw=28, c=1, k=8, repeat=0, layers=[(16, 6, 2, 0), "R", (16, 6, 2, 0), "R", ("d", 100), "R", ("d", 10)]),
    "f": dict(hw=32, c=3, k=7, repeat=5, layers=[(32, 3, 1, 0), "R", (32, 3, 1, 0), "R", (32, 2, 2, 0), (64, 3, 1, 0), "R", (64, 3, 1, 0), "R",
                                                 (64, 2, 2, 0), (128, 3, 1, 0), "R", (128, 3, 1, 0), "R", ("d", 10)]),
    "F": dict(hw=32, c=3, k=7, repeat=5, layers=[(64, 3, 1, 0), "R", (64, 3, 1, 0), "R", (64, 2, 2, 0), (64, 3, 1, 0), "R", (64, 3, 1, 0), "R",
                                                 (64, 2, 2, 0), (64, 3, 1, 0), "R", (64, 1, 1, 0), "R", (16, 1, 1, 0), "R", ("d", 10)]),
}
BIASED = ("A", "B", "C", "D", "f", "F")      # the paper's models have biases, the benchmark's configurations none


def listed():
    return [
        # one image through a small dense network: online latency, a chain of small dependent launches; and its garbling
        dict(name="mlp_b1_infer", kind="net", do="infer", net="mlp", batch=1, n_in=784, hidden=128, n_out=10, k=8, repeat=6, rule="ceil", digits="exact"),
        dict(name="mlp_b1_garble", kind="net", do="garble", net="mlp", batch=1, n_in=784, hidden=128, n_out=10, k=8, repeat=6, rule="ceil", digits="exact"),
        # one image through a small convolutional network of the paper: strides, biases, 9 primes, layers of 90 to 2 880 values
        dict(name="modelB_b1_infer", kind="net", do="infer", net="B", batch=1, rule="ceil", digits="exact"),
        # the paper's two CIFAR-sized networks, one image: the offline side of one, the online side of the other
        dict(name="modelF_b1_garble", kind="net", do="garble", net="F", batch=1, rule="ceil", digits="exact"),
        dict(name="modelf_b1_infer", kind="net", do="infer", net="f", batch=1, rule="ceil", digits="exact"),
        # a batch of 16 through LeNet-5: the main configuration, both sides
        dict(name="lenet_b16_garble", kind="net", do="garble", net="lenet", batch=16, rule="ceil", digits="exact"),
        dict(name="lenet_b16_infer", kind="net", do="infer", net="lenet", batch=16, rule="ceil", digits="exact"),
        # labels that pack into 128 bits: garble a batch of 4 and bring tables and output labels into the format that is stored and sent
        dict(name="lenet_floor_b4_ship", kind="net", do="ship", net="lenet", batch=4, rule="floor", digits="exact"),
        # one image of a VGG-sized network on the 12-prime base, layer by layer: the largest
        dict(name="vgg_b1_stream", kind="stream", batch=1, hw=32, width=64, k=12, repeat=5),
        # a large dense layer alone
        dict(name="dense_4096_b128", kind="linear", batch=128, hw=1, in_c=4096, out_c=4096, ksize=1, stride=1, pad=0, k=12, bias=False),
        # independent gates with mixed moduli, 4 M of them, both sides
        dict(name="proj_4m_garble", kind="proj", do="garble", gates=1 << 22, k=12),
        dict(name="proj_4m_eval", kind="proj", do="eval", gates=1 << 22, k=12),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["net", "net", "net", "net", "stream", "linear", "linear", "proj"])
    if kind == "net":
        do = rng.choice(["garble", "garble", "infer", "infer", "infer", "ship", "receive"])
        net = rng.choice(["mlp", "mlp", "mlp", "lenet", "lenet", "A", "B", "C", "D", "f", "F"])
        case = dict(kind=kind, do=do, net=net, rule="floor" if do in ("ship", "receive") else rng.choice(["ceil", "ceil", "ceil", "floor"]), digits="exact")
        if net == "mlp":
            case.update(n_in=_log(rng, 16, 1024), hidden=_log(rng, 10, 600), n_out=_log(rng, 2, 40), k=rng.choice([7, 8, 8, 9, 12]), repeat=rng.choice([0, 1, 4, 5, 6]))
        k = case.get("k") or CONVNETS[net]["k"]
        if k in REDUCED and rng.random() < 0.25:
            case["digits"] = "reduced"
        case["batch"] = _log(rng, 1, {"f": 1, "F": 1, "lenet": 16, "B": 32, "D": 32}.get(net, 64))
        limit = 8e9 if do in ("ship", "receive") else 20e9       # table bytes
        while case["batch"] > 1 and _table_bytes(_net(case), case) > limit:
            case["batch"] = case["batch"] * 2 // 3
        return case
    if kind == "stream":
        return dict(kind=kind, batch=rng.choice([1, 1, 2, 3]), hw=4 * rng.randint(2, 4), width=_log(rng, 4, 40), k=rng.choice([8, 12]), repeat=rng.randint(1, 5))
    if kind == "linear":
        case = dict(kind=kind, k=rng.choice([7, 8, 9, 12]), bias=rng.random() < 0.5)
        if rng.random() < 0.5:
            case.update(batch=_log(rng, 1, 128), hw=1, in_c=_log(rng, 24, 4096), out_c=_log(rng, 10, 4096), ksize=1, stride=1, pad=0)
        else:
            case.update(batch=_log(rng, 1, 32), hw=rng.randint(8, 32), in_c=rng.choice([1, 3, 6, _log(rng, 4, 128)]), out_c=_log(rng, 5, 256),
                        ksize=rng.choice([1, 2, 3, 3, 5]), stride=rng.choice([1, 1, 2]), pad=rng.choice([0, 1]))
        while case["batch"] > 1 and work(case)["flops"] > 2.3e12:
            case["batch"] //= 2
        return case
    return dict(kind=kind, do=rng.choice(["garble", "eval"]), gates=_log(rng, 500, 1 << 22), k=rng.choice([8, 12]))


# ---- networks in the format that GarbledNetwork and StreamedNetwork take -----------------------------------------
def _weights(gen, shape, lo, hi):
    return None if gen is None else gen.integers(lo, hi + 1, shape, dtype=np.int32)


class _Builder:
    """gen None: shapes only"""

    def __init__(self, gen, n_in, lo, hi, bias):
        self.gen, self.n, self.lo, self.hi, self.bias, self.layers = gen, n_in, lo, hi, bias, []

    def conv(self, h, c, out_c, ks, stride, pad):
        o = (h + 2 * pad - ks) // stride + 1
        L = dict(kind="conv", id=len(self.layers) + 1, in_h=h, in_w=h, in_c=c, out_c=out_c, kh=ks, kw=ks, stride=stride, pad=pad,
                 W=_weights(self.gen, (out_c, ks, ks, c), self.lo, self.hi), out_h=o, out_w=o, n_out=o * o * out_c)
        if self.bias and self.gen is not None:
            L["bias"] = _weights(self.gen, out_c, 16 * self.lo, 16 * self.hi)
        self.layers.append(L)
        self.n = L["n_out"]
        return o

    def dense(self, m):
        self.conv(1, self.n, m, 1, 1, 0)

    def relu(self, repeat):
        self.layers.append(dict(kind="relu", id=len(self.layers) + 1, n=self.n))
        if repeat:
            self.layers.append(dict(kind="scale", id=len(self.layers) + 1, n=self.n, repeat=repeat))

    def pool(self, h, c):
        self.layers.append(dict(kind="sumpool", id=len(self.layers) + 1, in_h=h, in_w=h, ch=c))
        self.n = (h // 2) ** 2 * c
        return h // 2


def _net(case, seed=None):
    gen = None if seed is None else np.random.Generator(np.random.Philox(key=[seed, 7]))
    if case["kind"] == "stream":
        k, n_in = case["k"], case["hw"] ** 2 * 3
        b, h, c = _Builder(gen, n_in, -16, 15, False), case["hw"], 3
        for width in (case["width"], 2 * case["width"], 4 * case["width"]):
            for _ in range(2):
                b.conv(h, c, width, 3, 1, 1)
                b.relu(case["repeat"])
                c = width
            h = b.pool(h, c)
        b.dense(4 * case["width"])
        b.relu(case["repeat"])
        b.dense(10)
    elif case["net"] == "mlp":
        k, n_in = case["k"], case["n_in"]
        b = _Builder(gen, n_in, -8, 7, False)
        b.dense(case["hidden"])
        b.relu(case["repeat"])
        b.dense(case["n_out"])
    else:
        spec = CONVNETS[case["net"]]
        k, n_in, h, c = spec["k"], spec["hw"] ** 2 * spec["c"], spec["hw"], spec["c"]
        b = _Builder(gen, n_in, -8, 7, case["net"] in BIASED)
        for L in spec["layers"]:
            if L == "R":
                b.relu(spec["repeat"])
            elif L == "P":
                h = b.pool(h, c)
            elif L[0] == "d":
                b.dense(L[1])
            else:
                h, c = b.conv(h, c, *L), L[0]
    digits = REDUCED[k] if case.get("digits") == "reduced" else DIGITS[k]
    return dict(primes=PRIMES[:k], digits=list(digits), batch=case["batch"], n_in=n_in, layers=b.layers)


def _seed_bytes(seed):
    return np.random.Generator(np.random.Philox(key=[seed, 3])).bytes(16)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _random_labels(ctx, labels, gen):
    """label digits uniform in Z_p, digits past lambda zero"""
    for i, t in enumerate(labels.tensors):
        if t is not None:
            p, lam = ctx.primes[i], ctx.lam(ctx.primes[i])
            t.copy_(torch.randint(0, p, t.shape, dtype=torch.uint8, device=ctx.device, generator=gen))
            if lam % 16:
                t[-1, :, lam % 16:] = 0


def prepare(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind in ("net", "stream"):
        net = _net(case, seed)
        ctx = Context(net["primes"], _seed_bytes(seed), net["digits"], LAMBDA_FLOOR if case.get("rule") == "floor" else LAMBDA_CEIL)
        x = torch.randint(0, 256, (net["batch"] * net["n_in"],), dtype=torch.int64, device=ctx.device, generator=gen)
        g = (GarbledNetwork if kind == "net" else StreamedNetwork)(ctx, net)
        state = dict(case=case, ctx=ctx, g=g, x=x)
        if kind == "stream":
            return state
        if case["do"] in ("ship", "receive"):
            state["packed"] = [None if t is None else torch.empty(ctx.tables_packed_bytes(l), dtype=torch.uint8, device=ctx.device)
                               for l, t in zip(g.layers, g.tables)]
            state["packed_out"] = torch.empty((ctx.k, g.sizes[-1], 16), dtype=torch.uint8, device=ctx.device)
        if case["do"] in ("infer", "receive"):
            g.garble()
        if case["do"] == "receive":
            _pack(state)
        return state
    if kind == "linear":
        ctx = Context(PRIMES[:case["k"]], _seed_bytes(seed), DIGITS[case["k"]])
        rng = np.random.Generator(np.random.Philox(key=[seed, 7]))
        hw, ks, in_c, out_c = case["hw"], case["ksize"], case["in_c"], case["out_c"]
        w = ctx.weights_prepare(rng.integers(-64, 64, (out_c, ks * ks * in_c), dtype=np.int32))
        bias = torch.as_tensor(rng.integers(-1024, 1024, out_c, dtype=np.int32)).to(ctx.device) if case["bias"] else None
        layer = Layer(DENSE if hw == 1 else CONV2D, 1, case["batch"], in_h=hw, in_w=hw, in_c=in_c, out_c=out_c, kh=ks, kw=ks, stride=case["stride"],
                      pad=case["pad"], weights=w, bias=bias)
        x = Labels(ctx, case["batch"] * hw * hw * in_c)
        _random_labels(ctx, x, gen)
        y = Labels(ctx, case["batch"] * ctx.layer_sizes(layer)[0])
        return dict(case=case, ctx=ctx, layer=layer, x=x, y=y)
    n, k = case["gates"], case["k"]
    ctx = Context(PRIMES[:k], _seed_bytes(seed), DIGITS[k])
    # moduli uniform over the base; how many gates each pair of moduli has depends on the case alone, their order on the seed
    pairs = np.random.Generator(np.random.Philox(key=[n, k])).integers(0, k * k, n, dtype=np.int16)
    np.random.Generator(np.random.Philox(key=[seed, 7])).shuffle(pairs)
    pb = ProjectionBatch(ctx, pairs // k, pairs % k)
    # one allocation behind the tables and one behind the output labels of every prime
    tables = torch.empty(pb.table_bytes, dtype=torch.uint8, device=ctx.device)
    per_q = [sum(G["count"] for G in pb.groups if G["qi"] == j) for j in range(k)]
    outs = {name: [torch.zeros(((ctx.lam(p) + 15) // 16, max(c, 1), 16), dtype=torch.uint8, device=ctx.device) for p, c in zip(ctx.primes, per_q)]
            for name in ("out0", "out")}
    at, at_q = 0, [0] * k
    for G in pb.groups:
        i, j, c = G["pi"], G["qi"], G["count"]
        size = G["table"].numel()
        G["table"] = tables[at:at + size]
        at += size
        for name in ("out0", "out"):
            G[name].tensors[j] = outs[name][j][:, at_q[j]:at_q[j] + c]
        at_q[j] += c
        _random_labels(ctx, G["in0"], gen)
        G["phi"].copy_(torch.randint(0, ctx.primes[j], G["phi"].shape, dtype=torch.uint8, device=ctx.device, generator=gen))
    if case["do"] == "eval":
        for G in pb.groups:
            ctx.encode(torch.randint(0, ctx.primes[G["pi"]], (G["count"],), dtype=torch.int64, device=ctx.device, generator=gen), G["in0"], G["act"])
        pb.garble()
    return dict(case=case, ctx=ctx, pb=pb, tables=tables, outs=outs)


def _pack(state):
    ctx, g = state["ctx"], state["g"]
    for layer, table, packed in zip(g.layers, g.tables, state["packed"]):
        if table is not None:
            ctx.tables_pack(layer, table, packed)
    ctx.labels_pack(g.zero[-1], state["packed_out"])


def run(state):
    case = state["case"]
    if case["kind"] == "linear":
        state["ctx"].eval_layer(state["layer"], state["x"], None, state["y"])
        return state["y"].tensors
    if case["kind"] == "proj":
        if case["do"] == "garble":
            state["pb"].garble()
            return dict(zero=state["outs"]["out0"], tables=state["tables"])
        state["pb"].evaluate()
        return state["outs"]["out"]
    g = state["g"]
    if case["kind"] == "stream":
        values, valid = g.run(state["x"])
        # label bundles of the network's output, and the tables of the last activation layer (the buffer's last tenant)
        last, n = len(g.layers) & 1, g.sizes[-1]
        return dict(values=values, valid=valid, zero=g.zero[last].slice(0, n).tensors, act=g.act[last].slice(0, n).tensors,
                    tables=g.table[:[t for t in g.layer_table_bytes if t][-1]])
    if case["do"] in ("garble", "ship"):
        g.garble()
        if case["do"] == "ship":
            _pack(state)
            return dict(packed=state["packed"], packed_out=state["packed_out"])
        return dict(zero=g.zero[-1].tensors, tables=g.tables)
    if case["do"] == "receive":
        for layer, packed, table in zip(g.layers, state["packed"], g.tables):
            if table is not None:
                state["ctx"].tables_unpack(layer, packed, table)
    g.encode(state["x"])
    g.evaluate()
    values, valid = g.decode()
    return dict(values=values, valid=valid, act=g.act[-1].tensors)


# ---- work ------------------------------------------------------------------------------------------------------
def _lam(m, rule="ceil"):
    n, v = 0, 1
    while v < 1 << 128:
        v, n = v * m, n + 1
    return n if rule == "ceil" or v == 1 << 128 else n - 1


def _gates(primes, digits, kind, repeat=1):
    """(rows, output modulus) of every projection gate over one value of an activation layer; modulus 0: rows of one digit"""
    k, n = len(primes), len(digits)
    m = [digits[0]] + [k * d for d in digits[1:]]

    def sign(first):
        return [(p, q) for p in primes[first:] for q in m] + [(m[j], m[j - 1]) for j in range(1, n)] + [(m[0], 2)]
    if kind == "relu":
        return sign(0) + [t for p in primes for t in ((p, p), (2, p), (2, 0))]
    return repeat * ([(2, p) for p in primes[1:]] + sign(1))


def _pitch(q, rule):
    return 4 * ((_lam(q, rule) + 3) // 4) if q else 4


def _activations(net):
    for L in net["layers"]:
        if L["kind"] in ("relu", "scale"):
            yield L["n"] * net["batch"], _gates(net["primes"], net["digits"], L["kind"], L.get("repeat", 1))


def _table_bytes(net, case):
    rule = case.get("rule", "ceil")
    return sum(E * sum(rows * _pitch(q, rule) for rows, q in gates) for E, gates in _activations(net))


def _conv_work(L, batch, primes, rule):
    """(bytes of the weights, multiply-adds on label digits as 2 operations each)"""
    K = L["kh"] * L["kw"] * L["in_c"]
    lam = sum(_lam(p, rule) for p in primes)
    return L["out_c"] * K * len(primes), 2.0 * batch * L["out_h"] * L["out_w"] * L["out_c"] * K * lam


# 32-bit lane operations of one hash: AES-128 as 160 look-ups and as many exclusive-ors, and a multiply and an addition for
# each of about 30 digits of the output label
HASH_OPS = 380.0


def work(case):
    kind, rule = case["kind"], case.get("rule", "ceil")
    if kind == "linear":
        primes, o = PRIMES[:case["k"]], (case["hw"] + 2 * case["pad"] - case["ksize"]) // case["stride"] + 1
        L = dict(kh=case["ksize"], kw=case["ksize"], in_c=case["in_c"], out_c=case["out_c"], out_h=o, out_w=o)
        w, ops = _conv_work(L, case["batch"], primes, "ceil")
        values = case["batch"] * (case["hw"] ** 2 * case["in_c"] + o * o * case["out_c"])
        return dict(bytes=w + values * sum(_lam(p) for p in primes), flops=ops)
    if kind == "proj":
        primes, n = PRIMES[:case["k"]], case["gates"]
        lam, mean_p = sum(_lam(p) for p in primes) / case["k"], sum(primes) / case["k"]
        if case["do"] == "garble":      # function table and input label read, rows and output label written
            return dict(bytes=n * (mean_p + lam + (mean_p + 1) * lam), flops=n * mean_p * HASH_OPS)
        return dict(bytes=n * 3 * lam, flops=n * HASH_OPS)
    net = _net(case)
    primes, batch = net["primes"], case["batch"]
    lam = sum(_lam(p, rule) for p in primes)
    ends = batch * lam * [L["n_out"] for L in net["layers"] if L["kind"] == "conv"][-1] + 8 * batch * net["n_in"]
    b_w = f_lin = rows_b = gates_b = n_rows = n_gates = 0.0
    for L in net["layers"]:
        if L["kind"] == "conv":
            w, ops = _conv_work(L, batch, primes, rule)
            b_w, f_lin = b_w + w, f_lin + ops
    for E, gates in _activations(net):
        rows_b += E * sum(rows * _pitch(q, rule) for rows, q in gates)
        gates_b += E * sum(_pitch(q, rule) for rows, q in gates)
        n_rows += E * sum(rows for rows, q in gates)
        n_gates += E * len(gates)
    garble, infer = (b_w + rows_b, f_lin + n_rows * HASH_OPS), (b_w + gates_b, f_lin + n_gates * HASH_OPS)
    packed = sum(E * sum(rows * (16 if q else 1) for rows, q in gates) for E, gates in _activations(net))
    b, f = {"garble": garble, "infer": infer, "ship": (b_w + packed, garble[1]), "receive": (b_w + 2 * gates_b, infer[1])}.get(
        case.get("do"), (b_w + rows_b + gates_b, garble[1] + infer[1]))
    return dict(bytes=b + ends, flops=f)


def tolerance(case):
    return "exact"      # labels, ciphertexts and decoded values are whole numbers
