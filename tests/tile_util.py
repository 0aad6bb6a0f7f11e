"""Which loops a head's contractions run on, asked of the library's own rules: tests of a loop say which one they mean, and
fail where a change of the rules has taken their sizes elsewhere."""
from paper_2505_24034_amd import binding


def loops(N, V, d, bf16=True, active=None):
    """(forward, dz, dH, dW): "64", "128" or "256", the tiles' edge; "256x128", "256x160", "256x256" or, forward only,
    "256x320" for the logits kernels of 256 vocabulary rows.  active: rows with gradient (all)"""
    r = binding._load_native()
    tiles_v = -(-V // 256)

    def logits(backward, n):
        edge = r.logits_tile(N, V, d, bf16, backward)
        if edge < 256:
            return str(edge)
        return "256x%d" % r.logits_width(tiles_v, n, d, min(256, tiles_v * -(-N // 128)), backward)

    n = N if active is None else active
    return logits(0, N), logits(1, n), str(r.store_tile(N, d, V, bf16)), str(r.store_tile(V, d, N, bf16))
