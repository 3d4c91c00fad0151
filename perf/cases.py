"""Performance cases: the solver's building blocks and short runs of its drivers, through the Python binding.

A case is one operation (`op`) on one game:
  gradient  both payoff products, A y and A^T x, of behavioural strategies (FP64, or the precision form in FP32);
  sbr       both players' smoothed best responses to a gradient, strategy and value (FP64 or the precision form);
  gap       the saddle gap of a strategy pair, on the host;
  steps     a restart from a checkpoint (iterates, products, scalars), `iters` driver iterations, and the iterates;
  solve     a whole solver call with an iteration budget (start-up and mu search included), and the iterates;
  cfr       a CFR+ run of `iters` iterations from scratch, and its averages and strategies.
Games are river endgames (`ranks` ranks of four cards, `board` of them public; every pair of the others is a hand) with
the bet rule `fracs` x pot + all-in and `raises` raises, or with the Libratus-style sizes (`fracs` = "libratus"), and
Leduc hold'em as a general game with an explicit payoff matrix.  Beliefs, strengths, strategies and gradients come from
the seed.

`exact` evaluates the same formulas densely in FP64 with torch, on a betting tree of its own.
"""
import math

import torch

from instances import LIBRATUS_RIVER, river
from instances.efg import leduc
from paper_1810_03063_amd import egt

C0 = dict(ranks=5, board=5, alpha=1.0, pot=100.0, stack=200.0, fracs="0.5 1", raises=2)
C1 = dict(ranks=13, board=5, alpha=0.5, pot=1000.0, stack=20000.0, fracs="0.5 1 2", raises=3)
C3 = dict(ranks=13, board=5, alpha=0.5, pot=1000.0, stack=20000.0, fracs="0.25 0.5 0.75 1 1.5 2 3", raises=4)
LIB = dict(ranks=13, board=5, alpha=0.5, pot=2100.0, stack=18950.0, fracs="libratus", raises=8)
WARM_STEPS = 6  # iterations before a checkpoint: the step size has settled


def listed():
    return [
        # the smallest products: a 105-hand toy endgame, what a test or a tutorial runs; launch latency
        dict(name="gradient_105h", op="gradient", dtype="f64", **C0),
        # the everyday endgame: 1081 hands, three bet sizes, 223 betting sequences
        dict(name="gradient_3sizes", op="gradient", dtype="f64", **C1),
        # the large endgame: eight bet sizes, 5938 betting sequences
        dict(name="gradient_8sizes", op="gradient", dtype="f64", **C3),
        # the same product in the precision form (matrix cores)
        dict(name="gradient_8sizes_f32", op="gradient", dtype="f32", **C3),
        # smoothed best responses with their values, as a caller of the single operations takes them
        dict(name="sbr_3sizes", op="sbr", dtype="f64", **C1),
        dict(name="sbr_8sizes", op="sbr", dtype="f64", **C3),
        dict(name="sbr_8sizes_f32", op="sbr", dtype="f32", **C3),
        # measuring the exploitability of a strategy pair on the Libratus-style tree
        dict(name="gap_libratus", op="gap", **LIB),
        # a solve under an iteration budget, EGT with mu balancing, on the everyday endgame
        dict(name="solve_3sizes", op="solve", variant="BAL", iters=64, **C1),
        # EGT/as iterations from a checkpoint on the large endgame: the headline solve's inner loop
        dict(name="steps_8sizes", op="steps", variant="AS", iters=4, **C3),
        # the comparison method: CFR+ from scratch on the everyday endgame
        dict(name="cfr_3sizes", op="cfr", iters=32, **C1),
        # a general game through the explicit payoff matrix
        dict(name="steps_leduc", op="steps", variant="BAL", iters=8, fracs="leduc", pot=2.0),
    ]


def draw(rng):
    op = rng.choice(["gradient", "gradient", "sbr", "sbr", "gap", "solve", "steps", "cfr"])
    ranks = rng.choice([5, 5, 6, 7, 8, 9, 10, 11, 12, 13])
    board = 5 if ranks == 13 else rng.choice([3, 4, 5])  # other boards give hand counts of other residues
    pot = round(100.0 * 2.0 ** rng.uniform(0, 4.5), 2)
    small = op in ("solve", "cfr")  # many iterations: trees up to the everyday endgame's
    if not small and rng.random() < 0.15:
        tree = dict(fracs="libratus", raises=8, stack=round(pot * rng.uniform(4, 20), 2))
    else:
        sizes = [0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0]
        k = rng.randint(1, 3 if small else 7)
        tree = dict(fracs=" ".join("%g" % f for f in sorted(rng.sample(sizes, k))), raises=rng.randint(0, 3 if small else 4),
                    stack=round(pot * rng.uniform(2, 20), 2))
    case = dict(op=op, ranks=ranks, board=board, alpha=rng.choice([0.5, 1.0]), pot=pot, **tree)
    if op in ("gradient", "sbr"):
        case["dtype"] = rng.choice(["f64", "f64", "f32"])
    elif op == "steps":
        case.update(variant=rng.choice(["AS", "BAL", "ALT"]), iters=rng.randint(1, 4))
    elif op == "solve":
        case.update(variant=rng.choice(["BAL", "ALT"]), iters=rng.randint(8, 64))
    elif op == "cfr":
        case["iters"] = rng.randint(4, 32)
    return case


# ---------------------------------------------------------------------------
# Games and inputs
# ---------------------------------------------------------------------------

def instance(case, seed):
    if case["fracs"] == "leduc":
        return leduc()
    lib = case["fracs"] == "libratus"
    return river("case", seed, case["ranks"], "int30" if case["ranks"] == 5 else "ranking_ties10", case["alpha"],
                 case["pot"], case["stack"], () if lib else [float(f) for f in case["fracs"].split()], case["raises"],
                 n_board=case["board"], abstraction=LIBRATUS_RIVER if lib else None)


class Tree:
    """One player's treeplex: information sets by height, a set's sequences contiguous."""

    def __init__(self, nodes):  # [(parent sequence or -1, number of actions)] with parents before children
        first, total = [], 0
        for _, na in nodes:
            first.append(total)
            total += na
        owner = [v for v, (_, na) in enumerate(nodes) for _ in range(na)]
        height, beta = [1] * len(nodes), [2.0] * len(nodes)
        for v in range(len(nodes) - 1, -1, -1):
            par = nodes[v][0]
            if par >= 0:
                height[owner[par]] = max(height[owner[par]], height[v] + 1)
                beta[owner[par]] += 2.0 * beta[v]
        order = sorted(range(len(nodes)), key=lambda v: height[v])
        self.new = [0] * total  # sequence as numbered by the caller -> row
        row, self.first, self.nact, self.beta, at = 0, [], [], [], {}
        for v in order:
            at[v] = len(self.first)
            self.first.append(row)
            self.nact.append(nodes[v][1])
            self.beta.append(beta[v])
            for a in range(nodes[v][1]):
                self.new[first[v] + a] = row + a
            row += nodes[v][1]
        self.n_seq = total
        self.parent = [self.new[nodes[v][0]] if nodes[v][0] >= 0 else -1 for v in order]
        depth_of_row, depth = [0] * total, [0] * len(order)
        for v in range(len(nodes)):
            par = nodes[v][0]
            depth[at[v]] = depth_of_row[self.new[par]] + 1 if par >= 0 else 0
            for a in range(nodes[v][1]):
                depth_of_row[self.new[first[v] + a]] = depth[at[v]]
        # sets of equal (height, action count), bottom-up, and of equal (depth, action count), top-down
        self.up, self.down = {}, {}
        for i, v in enumerate(order):
            self.up.setdefault((height[v], self.nact[i]), []).append(i)
            self.down.setdefault((depth[i], self.nact[i]), []).append(i)

    def groups(self, which, device):
        """[(sets, their rows [k, actions], their parents [k], beta [k, 1])] in order."""
        for key in sorted(which):
            sets = which[key]
            first = torch.tensor([self.first[i] for i in sets], device=device)
            yield (first[:, None] + torch.arange(key[1], device=device), torch.tensor([self.parent[i] for i in sets], device=device),
                   torch.tensor([self.beta[i] for i in sets], dtype=torch.float64, device=device)[:, None])


def betting(case):
    """Both players' trees and the terminals (kind, player-1 row or -1, player-2 row or -1, player 2's chips)."""
    pot, stack = case["pot"], case["stack"]
    lib = case["fracs"] == "libratus"
    nodes, count, terms = ([], []), [0, 0], []

    def amounts(p, c, bets):
        o = 1 - p
        if lib:
            fracs, allin = LIBRATUS_RIVER.fracs[p][min(bets, 3)], LIBRATUS_RIVER.allin[p][min(bets, 3)]
        else:
            fracs, allin = [float(f) for f in case["fracs"].split()], True
        base = pot + c[0] + c[1] + (c[o] - c[p])
        got = {min(c[o] + f * base, stack) for f in fracs} | ({stack} if allin else set())
        return sorted(a for a in got if a > c[o])

    def node(p, parent, na):
        nodes[p].append((parent, na))
        count[p] += na
        return count[p] - na

    def walk(c, p, bets, last):
        o = 1 - p
        facing = c[o] > c[p]
        acts = ["f", "c"] if facing else ["f", "k"] if lib and LIBRATUS_RIVER.open_fold[p] else ["k"]
        if not facing or (bets - 1 < case["raises"] and c[o] < stack):
            acts = acts + amounts(p, c, bets)
        first = node(p, last[p], len(acts))
        for i, a in enumerate(acts):
            nl = list(last)
            nl[p] = first + i
            if a == "f":
                if nl[o] < 0:
                    nl[o] = node(o, -1, 1)  # a fold before the opponent acted: its one-action pass
                terms.append((0, nl[0], nl[1], pot / 2 + c[0] if p == 0 else -(pot / 2 + c[1])))
            elif a == "c":
                terms.append((1, nl[0], nl[1], pot / 2 + c[o]))
            elif a == "k" and p == 1:
                terms.append((1, nl[0], nl[1], pot / 2 + c[0]))
            elif a == "k":
                walk(c, 1, bets, nl)
            else:
                walk([a if q == p else c[q] for q in (0, 1)], o, bets + 1, nl)

    walk([0.0, 0.0], 0, 0, [-1, -1])
    trees = [Tree(nodes[0]), Tree(nodes[1])]
    new = lambda p, s: trees[p].new[s] if s >= 0 else -1  # noqa: E731
    return trees, [(k, new(0, s), new(1, t), u) for k, s, t, u in terms]


def random_strategy(tree, n, ld, g):
    """A behavioural strategy in sequence form: softmax of normal logits at every (information set, hand)."""
    dev = "cuda"
    q = torch.exp(1.5 * torch.randn((tree.n_seq, ld), dtype=torch.float64, device=dev, generator=g))
    for rows, par, _ in tree.groups(tree.down, dev):
        w = q[rows]
        w = w / w.sum(1, keepdim=True)
        if int(par[0]) >= 0:
            w = w * q[par][:, None, :]
        q[rows] = w
    q[:, n:] = 0.0
    return q


def strategies(case, seed, trees, n, ld):
    g = torch.Generator(device="cuda").manual_seed(1000003 * (seed % 1000003) + 17)
    return [random_strategy(t, n, ld, g) for t in trees]


def gradients(case, seed, trees, n, ld, belief):
    """Gradients of the size the products have: chips times the player's own prior."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * (seed % 1000003) + 29)
    out = []
    for p, t in enumerate(trees):
        x = case["pot"] * torch.randn((t.n_seq, ld), dtype=torch.float64, device="cuda", generator=g)
        x[:, :n] *= belief[p]
        x[:, n:] = 0.0
        out.append(x)
    return out


def mu_of(case, n):
    return 0.05 * case["pot"] / n


def mu0_of(seed):
    return 0.02 * (1.0 + (seed % 97) / 97.0)


def slot_beliefs(inst):
    """Both priors with the hands in ascending strength (ties in the given order)."""
    order = torch.argsort(torch.from_numpy(inst.strength), stable=True)
    return [torch.from_numpy(inst.belief[p])[order].cuda() for p in (0, 1)], order


def prepare(case, seed):
    inst = instance(case, seed)
    G = egt.GeneralGame(inst) if case["fracs"] == "leduc" else egt.Game(inst)
    S = dict(case=case, game=G)
    op = case["op"]
    f32 = case.get("dtype") == "f32"
    if op in ("gradient", "gap"):
        trees, _ = betting(case)
        xy = strategies(case, seed, trees, G.n, G.ld)
        S["x"], S["y"] = [v.float() if f32 else v for v in xy]
        if op == "gradient":
            S["out"] = [G.empty(p, dtype=S["x"].dtype) for p in (0, 1)]
            if f32:  # the precision form's tables are built once per game
                egt.gradient_mixed(G, 0, S["y"], S["out"][0])
    elif op == "sbr":
        trees, _ = betting(case)
        b, _ = slot_beliefs(inst)
        S["g"] = [v.float() if f32 else v for v in gradients(case, seed, trees, G.n, G.ld, b)]
        S["q"] = [torch.zeros_like(v) for v in S["g"]]
        S["value"] = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in (0, 1)]
    elif op == "steps":
        mu0 = (mu0_of(seed), mu0_of(seed)) if case["fracs"] == "leduc" else None
        st = egt.State(G, variant=case["variant"], mu0=mu0)
        for _ in range(WARM_STEPS):
            st.step()
        S["state"], S["from"] = st, st.get()
        S["from"]["ay"], S["from"]["atx"] = st.products()
    return S


def run(S):
    case, G = S["case"], S["game"]
    op = case["op"]
    f32 = case.get("dtype") == "f32"
    if op == "gradient":
        f = egt.gradient_mixed if f32 else egt.gradient
        return {"ay": f(G, 0, S["y"], S["out"][0]), "atx": f(G, 1, S["x"], S["out"][1])}
    if op == "sbr":
        f = egt.smoothed_br_mixed if f32 else egt.smoothed_br
        mu = mu_of(case, G.n)
        for p in (0, 1):
            f(G, p, S["g"][p], mu, S["q"][p], S["value"][p])
        return {"q": S["q"], "value": S["value"]}
    if op == "gap":
        gap, br_max, br_min = egt.saddle_gap(G, S["x"], S["y"])
        return {"gap": gap, "br_max_y": br_max, "br_min_x": br_min}
    if op == "steps":
        st, f = S["state"], S["from"]
        st.set(f["x"], f["y"], f["mu_x"], f["mu_y"], f["tau"], f["iters"], f["ay"], f["atx"])
        for _ in range(case["iters"]):
            st.step()
        r = st.get()
        return {"x": r["x"], "y": r["y"], "mu_x": r["mu_x"], "mu_y": r["mu_y"]}
    if op == "solve":
        res, st = egt.solve(G, keep_state=True, variant=case["variant"], max_iters=case["iters"], eps=1e-12)
        r = st.get()
        st.close()
        return {"x": r["x"], "y": r["y"], "gap": res["gap"], "value": res["value_p1"]}
    c = egt.Cfr(G, "CFR_PLUS")
    c.step(case["iters"])
    r = c.get()
    c.close()
    return {k: r[k] for k in ("x_avg", "y_avg", "x", "y")}


def work(case):
    """Each operand in and each result out once (iterations: both players' iterates and products in and out once)."""
    if case["fracs"] == "leduc":
        n, seqs, terms = 1, [336, 336], 966
    else:
        trees, z = betting(case)
        cards = 4 * case["ranks"] - case["board"]
        n, seqs, terms = cards * (cards - 1) // 2, [t.n_seq for t in trees], len(z)
    esz = 4 if case.get("dtype") == "f32" else 8
    v = esz * n * sum(seqs)  # one vector of each player
    product, response = 2 * 10 * n * terms, 40 * n * sum(seqs)  # both players'
    op, iters = case["op"], case.get("iters", 1)
    if op == "gradient":
        return {"bytes": 2 * v, "flops": product}
    if op == "sbr":
        return {"bytes": 2 * v, "flops": response}
    if op == "gap":
        return {"bytes": v, "flops": product + response / 10}
    if op == "cfr":
        return {"bytes": iters * 6 * v, "flops": iters * (product + response / 4)}
    return {"bytes": iters * 4 * v, "flops": iters * (1.5 * product + 2.5 * response)}


# ---------------------------------------------------------------------------
# The same results in FP64, densely
# ---------------------------------------------------------------------------

class Dense:
    """The game of a case as dense matrices, and the paper's formulas on it."""

    def __init__(self, case, inst):
        self.dev = dev = "cuda" if torch.cuda.is_available() else "cpu"
        f64 = torch.float64
        if case["fracs"] == "leduc":
            self.n, self.ld = 1, 32
            self.trees = [Tree([(s[0], s[1]) for s in inst.infosets[p]]) for p in (0, 1)]
            A = torch.zeros((self.trees[0].n_seq, self.trees[1].n_seq), dtype=f64)
            for s, t, v in inst.entries:
                A[self.trees[0].new[s], self.trees[1].new[t]] += v
            self.A = A.to(dev)
            return
        self.A = None
        self.trees, terms = betting(case)
        order = torch.argsort(torch.from_numpy(inst.strength), stable=True)
        cards = torch.from_numpy(inst.hand_cards).long()[order].to(dev)
        strength = torch.from_numpy(inst.strength).long()[order].to(dev)
        self.n = n = cards.shape[0]
        self.ld = (n + 31) // 32 * 32
        share = (cards[:, None, :, None] == cards[None, :, None, :]).any(-1).any(-1)
        compat = (~share).to(f64)
        self.M = [compat, compat * torch.sign((strength[None, :] - strength[:, None]).to(f64))]
        self.b = [torch.from_numpy(inst.belief[p])[order].to(dev) for p in (0, 1)]
        self.Z = self.b[0] @ compat @ self.b[1]
        self.terms = []  # per kind: rows of player 1, of player 2, chips
        for kind in (0, 1):
            z = [t for t in terms if t[0] == kind]
            self.terms.append([torch.tensor([t[i] for t in z], device=dev) for i in (1, 2)]
                              + [torch.tensor([t[3] for t in z], dtype=f64, device=dev)])

    def product(self, p, v):
        """Player p's gradient at the opponent's strategy v."""
        out = torch.zeros((self.trees[p].n_seq, self.ld), dtype=torch.float64, device=self.dev)
        if self.A is not None:
            out[:, 0] = (self.A if p == 0 else self.A.T) @ v[:, 0]
            return out
        o, n = 1 - p, self.n
        for kind in (0, 1):
            rows, chips = self.terms[kind][:2], self.terms[kind][2]
            reach = v[rows[o].clamp(min=0), :n].clone()
            reach[rows[o] < 0] = 1.0
            part = (reach * self.b[o]) @ self.M[kind].T * chips[:, None]
            part *= -1.0 if kind == 1 and p == 1 else 1.0
            # at most a few terminals of one kind end at the same own sequence: add them rank by rank
            part, own = part[rows[p] >= 0], rows[p][rows[p] >= 0]
            srt = torch.argsort(own, stable=True)
            own, part = own[srt], part[srt]
            start = torch.searchsorted(own, own)
            rank = torch.arange(len(own), device=self.dev) - start
            for r in range(int(rank.max()) + 1 if len(own) else 0):
                out[own[rank == r], :n] += part[rank == r]
        out[:, :n] *= self.b[p] / self.Z
        return out

    def up(self, p, g, weight):
        """Bottom-up: weight(g~ [sets, actions, hands], beta) gives values and local strategies."""
        t = self.trees[p]
        gt, loc, total = g[:, : self.n].clone(), torch.zeros_like(g[:, : self.n]), 0.0
        for rows, par, beta in t.groups(t.up, self.dev):
            val, w = weight(gt[rows], beta, rows)
            loc[rows] = w
            inner = par >= 0
            gt.index_put_((par[inner],), val[inner], accumulate=True)
            total = total + val[~inner].sum()
        return total, loc

    def down(self, p, loc):
        t = self.trees[p]
        q = torch.zeros((t.n_seq, self.ld), dtype=torch.float64, device=self.dev)
        for rows, par, _ in t.groups(t.down, self.dev):
            w = loc[rows]
            q[rows, : self.n] = w * q[par][:, None, : self.n] if int(par[0]) >= 0 else w
        return q

    def sbr(self, p, g, mu):
        def weight(x, beta, rows):
            m = x.min(1, keepdim=True).values
            temp = mu * beta[:, :, None]
            w = torch.exp((m - x) / temp)
            s = w.sum(1, keepdim=True)
            return (m - temp * torch.log(s) + temp * math.log(x.shape[1]))[:, 0], w / s

        val, loc = self.up(p, g, weight)
        return self.down(p, loc), val

    def best(self, p, g):
        return self.up(p, g, lambda x, beta, rows: (x.min(1).values, torch.zeros_like(x)))[0]

    def uniform(self, p):
        return self.down(p, self.up(p, torch.zeros((self.trees[p].n_seq, self.ld), dtype=torch.float64, device=self.dev),
                                    lambda x, beta, rows: (x[:, 0], torch.full_like(x, 1.0 / x.shape[1])))[1])

    def gap(self, x, y):
        br_min, br_max = self.best(0, self.product(0, y)), -self.best(1, -self.product(1, x))
        return br_max - br_min, br_max, br_min

    def start(self, mu0):
        x_w = self.uniform(0)
        a = self.product(1, x_w)
        mu = mu0
        if mu is None:
            top = max(float(a.abs().max()), float(self.product(0, self.uniform(1)).abs().max()))
            mu = 1e-3 * top / max(max(t.beta) for t in self.trees)
        while True:
            y = self.sbr(1, -a, mu)[0]
            x = self.sbr(0, self.product(0, y), mu)[0]
            if mu0 is not None or self.egv(x, y, [mu, mu]) >= 0:
                return [x, y], [mu, mu]
            mu *= 2.0

    def egv(self, x, y, mu):
        return self.sbr(0, self.product(0, y), mu[0])[1] + self.sbr(1, -self.product(1, x), mu[1])[1]

    def step(self, z, mu, tau, p, search):
        """One step focused on p (Algorithm 2; with `search` Algorithm 4's halvings)."""
        o, sg = 1 - p, (1.0, -1.0)
        g = sg[p] * self.product(p, z[o])
        bar = self.sbr(p, g, mu[p])[0]
        while True:
            hat = (1 - tau) * z[p] + tau * bar
            other = self.sbr(o, sg[o] * self.product(o, hat), mu[o])[0]
            new, mu_new = [None, None], list(mu)
            new[o] = (1 - tau) * z[o] + tau * other
            prox = self.sbr(p, g + tau / (1 - tau) * sg[p] * self.product(p, other), mu[p])[0]
            new[p] = (1 - tau) * z[p] + tau * prox
            mu_new[p] = (1 - tau) * mu[p]
            if not search or self.egv(new[0], new[1], mu_new) >= 0:
                return new, mu_new, tau
            tau *= 0.5

    def iterate(self, variant, iters, mu0=None):
        z, mu = self.start(mu0)
        tau = 0.5
        for t in range(iters):
            p = t % 2 if variant == "ALT" else (0 if mu[0] > mu[1] else 1)
            if variant != "AS":
                tau = 2.0 / (t + 3.0)
            z, mu, tau = self.step(z, mu, tau, p, variant == "AS")
        return z, mu

    def cfr_plus(self, iters):
        z = [self.uniform(0), self.uniform(1)]
        loc = [torch.cat([torch.full((na, self.n), 1.0 / na, dtype=torch.float64, device=self.dev) for na in t.nact]) for t in self.trees]
        regret = [torch.zeros_like(v) for v in loc]
        avg, total = [v.clone() for v in z], 0.0
        for t in range(1, iters + 1):
            total += t
            avg = [a + (t / total) * (v - a) for a, v in zip(avg, z)]
            for p in (0, 1):
                g = (1.0, -1.0)[p] * self.product(p, z[1 - p])
                top = g[:, : self.n].abs().max()

                def weight(x, beta, rows):
                    val = (loc[p][rows] * x).sum(1, keepdim=True)
                    r = val - x
                    r = torch.where(r.abs() <= 1e-12 * (val.abs() + x.abs() + top), 0.0, r)
                    R = (regret[p][rows] + r).clamp(min=0.0)
                    regret[p][rows] = R
                    s = R.sum(1, keepdim=True)
                    return val[:, 0], torch.where(s > 0, R / torch.where(s > 0, s, 1.0), 1.0 / x.shape[1])

                loc[p] = self.up(p, g, weight)[1]
                z[p] = self.down(p, loc[p])
        return avg, z


def exact(case, seed):
    inst = instance(case, seed)
    D = Dense(case, inst)
    op = case["op"]
    if op in ("gradient", "gap"):
        x, y = strategies(case, seed, D.trees, D.n, D.ld)
        if case.get("dtype") == "f32":
            x, y = x.float().double(), y.float().double()
        if op == "gradient":
            return {"ay": D.product(0, y), "atx": D.product(1, x)}
        gap, br_max, br_min = D.gap(x, y)
        return {"gap": float(gap), "br_max_y": float(br_max), "br_min_x": float(br_min)}
    if op == "sbr":
        g = gradients(case, seed, D.trees, D.n, D.ld, D.b)
        got = [D.sbr(p, v.float().double() if case["dtype"] == "f32" else v, mu_of(case, D.n)) for p, v in enumerate(g)]
        return {"q": [q for q, _ in got], "value": [v.reshape(1) for _, v in got]}
    if op == "steps":
        z, mu = D.iterate(case["variant"], WARM_STEPS + case["iters"], mu0_of(seed) if case["fracs"] == "leduc" else None)
        return {"x": z[0], "y": z[1], "mu_x": float(mu[0]), "mu_y": float(mu[1])}
    if op == "solve":
        z, _ = D.iterate(case["variant"], case["iters"])
        return {"x": z[0], "y": z[1], "gap": float(D.gap(z[0], z[1])[0]),
                "value": -float((z[0] * D.product(0, z[1])).sum())}
    avg, z = D.cfr_plus(case["iters"])
    return {"x_avg": avg[0], "y_avg": avg[1], "x": z[0], "y": z[1]}
