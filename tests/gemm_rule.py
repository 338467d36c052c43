"""Which kernel a canonical GEMM runs on (a mirror of the library's rule on a GPU of 256 CUs), so that a test can say that
it reaches the kernel it is about."""

FULL, TRAIL, LEAD = 0, 1, 2  # all of K; keys up to the tile's queries (P.V, dQ); queries from the tile's keys on (dK, dV)


def split_config(m, n, k, batch=1, kmode=FULL, kwin=0, kseg=0, cus=256):
    """(row groups, K blocks) of the split kernel, or None for the general (or short-contraction) kernels."""
    if m < 16 or n < 16 or k < 8:
        return None
    chunks = -(-k // 32)

    def fits(rows, cols):
        return -(-m // rows) * -(-n // cols) * batch <= cus

    if kmode == FULL and kseg == 0:
        if chunks >= 48 and fits(16, 16):
            return (1, 4)
        if chunks >= 2 and fits(16, 32):
            return (1, 2)
    if fits(16, 64):
        return (1, 1)
    if kmode == LEAD and kseg == 0 and 0 < 4 * kwin <= k and chunks >= 128:
        return None
    return (2, 1) if fits(32, 64) else None


def attention_configs(batch, heads, kv_heads, seq, head_dim, window):
    """Configurations of a block's causally skipping products: P.V and dQ, and dK and dV."""
    g = heads // kv_heads
    seg = g == 1 or seq % 128 == 0
    return (split_config(seq, head_dim, seq, batch * heads, TRAIL, window),
            split_config(seq, head_dim, g * seq, batch * kv_heads, LEAD if seg else FULL, window if seg else 0,
                         seq if seg and g > 1 else 0))


def general_batch(m, n):
    """A batch of m x n outputs that no split takes."""
    return 256 // (-(-m // 32) * -(-n // 64)) + 1
