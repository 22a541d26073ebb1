"""Hardware-aware mixed-precision selection (Section 3.4): choose a bit width per layer group by an integer linear
programme that minimises the summed sensitivity subject to limits on model size, bit operations and latency --
with the latency table measured on this GPU by the library's own kernels.

    minimise    sum_i Omega_i^(b_i)
    subject to  sum_i M_i^(b_i) <= size limit,  sum_i G_i^(b_i) <= BOPS limit,  sum_i Q_i^(b_i) <= latency limit

M_i is the size of layer i at b_i bits, G_i = b_w b_a MAC_i its bit operations (weights and activations of a layer share
one width), Q_i its measured latency.  Any subset of the limits may be given.  The sensitivities Omega are an input:
the paper takes a Hessian-based perturbation measured on training data, which this repository does not have;
`quantization_perturbation` gives the data-free part of that metric (the squared weight perturbation) as a stand-in.
On MI355X there is no INT4 matrix instruction, so 4 bits buy bytes and not multiply-accumulates: the measured Q_i
differ from the BOPS model layer by layer, which is exactly what the latency constraint is for.
"""
import numpy as np

from .binding import hawq_net_layer_info, hawq_net_num_layers


def group_of(name):
    """Layers that must share a bit width form a group: a transition convolution goes with its block's first one."""
    return name[:-2] + "c1" if name.endswith(".ds") else name


def layer_costs(arch, image_hw=224, num_classes=1000, choices=(4, 8)):
    """Per group: weight bytes M and bit operations G for every bit choice (conv1 and fc are fixed at 8 bits and
    appear with identical entries).  Returns (group names in network order, M [G, B] bytes, G [G, B] bit operations)."""
    names, M, Gb = [], {}, {}
    for i in range(hawq_net_num_layers(arch)):
        f = hawq_net_layer_info(arch, image_hw, num_classes, i)
        g = group_of(f["name"])
        if g not in M:
            names.append(g)
            M[g] = np.zeros(len(choices))
            Gb[g] = np.zeros(len(choices))
        params = f["K"] * f["R"] * f["S"] * f["C"]
        macs = params * f["P"] * f["Q"]
        for j, b in enumerate(choices):
            bb = 8 if f["name"] in ("conv1", "fc") else b
            M[g][j] += params * bb / 8.0
            Gb[g][j] += float(bb) * bb * macs
    return names, np.array([M[g] for g in names]), np.array([Gb[g] for g in names])


def quantization_perturbation(W, bits):
    """|| Q(W) - W ||^2 with the converter's per-channel symmetric quantiser: the data-free factor of the
    second-order sensitivity metric (stand-in when no Hessian information is available)."""
    from .convert import quantize_weights
    q, S = quantize_weights(W, bits)
    return float(np.sum((np.asarray(W, dtype=np.float64) - q * S.reshape(-1, 1, 1, 1)) ** 2))


def solve(omega, size=None, bops=None, latency=None, size_limit=None, bops_limit=None, latency_limit=None, fixed=None):
    """Exact solution of the selection problem.  omega, size, bops, latency: [L, B] arrays (row = layer group, column =
    bit choice); a limit of None drops that constraint.  fixed: {row: column} choices imposed beforehand.
    Returns (choice [L] column indices, objective) or raises ValueError if the limits cannot be met.

    No limit is exceeded by more than the rounding of its sum.  The solver itself takes a choice within its tolerance of a limit for one that holds it; such a
    choice is excluded and the problem solved again, sixteen times at most.  Where equal rows make more of them than that, the
    limit is lowered by that tolerance (doubled as long as it takes): the result then still holds every limit, and only a
    choice within a few parts in 10^9 of one may have been passed over."""
    from scipy.optimize import Bounds, LinearConstraint, milp
    omega = np.asarray(omega, dtype=np.float64)
    L, B = omega.shape
    tolerance = 1e-6                                     # of the solver, on a row's sum
    A, lo, hi, limits = [], [], [], []                   # limits: [table, limit, row of A, margin below it]
    for i in range(L):                                   # exactly one choice per group
        row = np.zeros(L * B)
        row[i * B:(i + 1) * B] = 1
        A.append(row); lo.append(1); hi.append(1)
    for tab, lim in ((size, size_limit), (bops, bops_limit), (latency, latency_limit)):
        if lim is None:
            continue
        if tab is None:
            raise ValueError("a limit needs its cost table")
        tab = np.asarray(tab, dtype=np.float64).reshape(-1)
        if not np.isfinite(tab).all():
            raise ValueError("a cost table must be finite")
        limits.append([tab.reshape(L, B), float(lim), len(A), tolerance])
        # the tolerance is absolute: small tables are scaled up to a largest entry of 1000, large ones stay as they are
        scale = max(1.0, 1e3 / max(np.abs(tab).max(), 1e-30))
        A.append(tab * scale); lo.append(-np.inf); hi.append(float(lim) * scale)
    ub = np.ones(L * B)
    lb = np.zeros(L * B)
    for i, j in (fixed or {}).items():
        lb[i * B + j] = 1
    rows, singly = len(A), 16
    while True:
        res = milp(c=omega.reshape(-1), integrality=np.ones(L * B), bounds=Bounds(lb, ub),
                   constraints=LinearConstraint(np.array(A), np.array(lo), np.array(hi)))
        if not res.success:
            raise ValueError("bit selection infeasible under the given limits: " + str(res.message))
        choice = np.rint(res.x).reshape(L, B).argmax(axis=1)
        over = [l for l in limits if l[0][np.arange(L), choice].sum() > l[1] + 1e-12 * abs(l[1])]
        if not over:
            break
        if singly > 0:
            singly -= 1
            row = np.zeros((L, B))                       # anything but this choice
            row[np.arange(L), choice] = 1
            A.append(row.reshape(-1)); lo.append(0); hi.append(L - 1)
        else:
            del A[rows:], lo[rows:], hi[rows:]           # (the lower limit excludes those too)
            for l in over:
                hi[l[2]] -= l[3]
                l[3] *= 2
    return choice, float(omega[np.arange(L), choice].sum())


def least_cost(table, fixed=None):
    """The least sum that any choice under `fixed` ({row: column}) has in a cost table [L, B]: a limit from there on can be met."""
    table = np.asarray(table, dtype=np.float64)
    return float(sum(table[i, fixed[i]] if i in (fixed or {}) else table[i].min() for i in range(len(table))))


def share_block_time(times, work, stored):
    """Time of a block that runs as one launch, per bit choice, as its groups' shares: {group: [B]}.  The launch computes on bytes at
    every width and keeps what lies between its convolutions on the chip, so a width changes its time only where it changes how
    the block's input or output is stored.  What every choice takes is dealt to the block's groups by their work ({group:
    multiply-accumulates}), what one takes beyond that in equal parts to `stored`, the groups whose widths set that storage."""
    times = np.asarray(times, dtype=np.float64)
    least, total = times.min(), float(sum(work.values()))
    out = {g: np.zeros(len(times)) for g in list(work) + list(stored)}
    for g in work:
        out[g] += least * work[g] / total
    for g in stored:
        out[g] += (times - least) / len(stored)
    return out


def measure_group_latencies(net_by_choice, batch, image, repeats=5):
    """Measured latency table Q [G, B] in milliseconds for one batch size: net_by_choice maps a bit choice to a
    HawqNet in which every selectable group runs at that width; the per-launch device times of the library's timed
    forward are summed per group (a transition convolution into its block's first group; conv1 carries the fused max
    pool); the time of a block that runs as one launch goes to the groups as share_block_time has it, with the first
    convolution of the next block among those whose width sets its storage.  Returns (group names, Q)."""
    import torch
    names = None
    cols, blocks = [], []
    for b in sorted(net_by_choice):
        hn = net_by_choice[b]
        ws = torch.empty(hn.workspace_bytes(batch), dtype=torch.uint8, device="cuda")
        logits = torch.empty((batch, hn.num_classes), dtype=torch.int32, device="cuda")
        for _ in range(2):
            hn.hawq_forward_resnet(image, batch, logits, ws)
        per = np.median(np.array([hn.hawq_forward_resnet_timed(image, batch, logits, ws) for _ in range(repeats)]), axis=0)
        steps = [hn.step_output(batch, s) for s in range(hn.num_steps())]
        acc, order, idle = {}, [], set()
        for s, st in enumerate(steps):
            nm = st["name"]
            if hn.step_cost(batch, s)[0] == 0:
                idle.add(nm)                             # (no convolution, or computed in the launch at a later step)
            g = "conv1" if nm == "pool" else ("fc" if nm == "avgpool" else group_of(nm))
            if g not in acc:
                acc[g] = 0.0
                order.append(g)
            acc[g] += float(per[s])
        joined = {}                                      # block: (storage of its input, of its output, the group that reads that)
        for s, st in enumerate(steps):
            blk = st["name"][:-3]
            if st["name"] == blk + ".c1" and st["name"] in idle and blk + ".c2" in idle:
                last = max(i for i, o in enumerate(steps) if o["name"].startswith(blk + "."))
                joined[blk] = (steps[s - 1]["dtype"], steps[last]["dtype"], group_of(steps[last + 1]["name"]))
        if names is None:
            names = order
        cols.append(acc)
        blocks.append(joined)
    cost_names, _, ops = layer_costs(hn.arch, hn.image_hw, hn.num_classes, (8,))
    costs = dict(zip(cost_names, ops[:, 0]))
    Q = {g: np.array([acc[g] for acc in cols]) for g in names}
    extra = {g: np.zeros(len(cols)) for g in names}
    for blk in sorted(set().union(*blocks)):
        work = {g: costs[g] for g in names if g.startswith(blk + ".")}
        times = sum(Q[g] for g in work)
        first, here = blk + ".c1", [j for j in range(len(cols)) if blk in blocks[j]]
        inputs, outputs = ({blocks[j][blk][i] for j in here} for i in (0, 1))
        stored = ([first] if len(inputs) > 1 else []) + ([blocks[here[0]][blk][2]] if len(outputs) > 1 else [])
        shares = share_block_time(times[here], work, stored or [first])
        for g in work:
            Q[g][here] = 0                               # (a choice with separate launches keeps their times)
        for g in shares:
            extra[g][here] += shares[g]
    return names, np.array([Q[g] + extra[g] for g in names])
