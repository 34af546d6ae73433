"""The rules by which a bf16 call of the prefill kernel takes its variant, from what the map says of itself on the host."""
import numpy as np


def tiles_read(tm, head_class):
    """Key tiles of one KV head that a launch for these classes reads: runs of visited tiles of the prompt, of free keys and of text keys."""
    seen = None
    for c in sorted(set(int(x) for x in head_class)):
        for m in range(tm.n_q_tiles):
            states = tm.walked(c, m)[0] != 0
            seen = states if seen is None else seen | states
    n0 = tm.key_order()[1]
    total = 0
    for lo, hi in ((0, n0), (n0, tm.n_k_tiles), (tm.n_k_tiles, len(seen))):
        at = np.flatnonzero(seen[lo:hi])
        total += at[-1] - at[0] + 1 if len(at) else 0
    return int(total)


def transposed_values(d, steps, tiles):
    """V is transposed ahead of the launch: tiles of all KV heads that are walked at least so many times on average."""
    line = (22 if d == 128 else 0) if tiles <= 256 else 32 if d == 128 else 4 if tiles <= 4096 else 10
    return steps >= line * tiles


def variant(tm, head_class, n_kv, d, n_wgs=256):
    """(steps of two tiles, V transposed ahead, steps per tile, tiles, cut units) of a call with all heads of these classes."""
    G = len(head_class) // n_kv
    plan, shares = tm.pair_plan(G), tm.share_plan(G, n_wgs)
    steps, tiles = plan["unit_tiles"], tiles_read(tm, head_class) * n_kv
    n_shares = n_wgs if shares["n_parts"] else 0
    return (d == 64 and steps >= 12 * max(plan["n_units"], n_shares), transposed_values(d, steps, tiles), steps / tiles, tiles, shares["n_cut_units"])
