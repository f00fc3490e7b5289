"""Which way a batch goes through the attention calls, and how many records a segment (request, KV head) leaves: the rules
of csrc/pkv_kernels.h and of the stream pass once more, so that a test can say which kernels its shapes reach and fails when a rule
moves them elsewhere.  tests/test_routes.py holds the host's rules here against the library's own."""
import numpy as np

GROUPS = 256   # workgroups of a full launch
BLOCK = 16     # tokens


def group_waves(dim):
    return 4 if dim == 256 else 8


def full_waves(dim):
    return GROUPS * group_waves(dim)


def short_blocks(segments, dim, fp8=False):
    """Longest segment of a batch that is cut along its segments."""
    small = segments <= 64 and 2 * BLOCK * dim * (1 if fp8 else 2) >= 8192
    return (3 if small else 6) * group_waves(dim)


def row_blocks(dim):
    """The most blocks that go by rows."""
    return 2 * full_waves(dim)


def leaves(segments, max_blocks, G, dim, fp8=False):
    """The host's choice: "none", "rows", "few" or "many"."""
    if segments <= GROUPS and max_blocks <= short_blocks(segments, dim, fp8):
        return "none"
    if segments > 64 or segments < 32 or G * dim > 64:
        return "many"
    return "rows" if segments * max_blocks <= row_blocks(dim) else "few"


def blocks_of(w):
    return (np.asarray(w.context_lens, dtype=np.int64) + BLOCK - 1) // BLOCK


def host_route(w, max_context_len=0, fp8=False):
    bound = max_context_len or w.max_blocks_per_seq * w.block_size
    return leaves(w.num_seqs * w.num_kv_heads, (bound + BLOCK - 1) // BLOCK, w.num_q_heads // w.num_kv_heads, w.head_dim, fp8)


def route(w, max_context_len=0, fp8=False):
    """What becomes of the batch, with the device's part of the choice: "whole" (cut along its segments), "dealt" (by rows,
    less than a block for each wavefront), "rows" (by rows) or "records" (workgroups' records)."""
    host, segments, nb = host_route(w, max_context_len, fp8), w.num_seqs * w.num_kv_heads, blocks_of(w)
    if host == "none" or (segments <= GROUPS and nb.max() <= short_blocks(segments, w.head_dim, fp8)):
        return "whole"
    T = int(nb.sum()) * w.num_kv_heads
    if host in ("rows", "few") and T <= row_blocks(w.head_dim):
        return "dealt" if T < full_waves(w.head_dim) else "rows"
    return "records"


def records(w):
    """Workgroups that share each segment of a batch of workgroups' records, 1 where one finishes it; requests with no tokens left out."""
    nb = blocks_of(w)
    T, group = int(nb.sum()) * w.num_kv_heads, group_waves(w.head_dim)
    W = min(T, full_waves(w.head_dim))
    starts = np.arange(W + 1, dtype=np.int64) * T // W
    lengths = np.repeat(nb[nb > 0], w.num_kv_heads)
    first = np.cumsum(lengths) - lengths
    owner = lambda pos: (np.searchsorted(starts, pos, side="right") - 1) // group
    return (owner(first + lengths - 1) - owner(first) + 1).tolist()
