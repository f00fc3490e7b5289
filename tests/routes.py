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


def leaves_records(segments, max_blocks, dim, fp8=False):
    """By the bounds: may workgroups share segments, so that there is a reduce pass?"""
    return segments > GROUPS or max_blocks > short_blocks(segments, dim, fp8)


def blocks_of(w):
    return (np.asarray(w.context_lens, dtype=np.int64) + BLOCK - 1) // BLOCK


def route(w, max_context_len=0, fp8=False):
    """What becomes of the batch: "whole" (cut along its segments, as the bounds say), "whole on the device" (as it finds from
    the lengths) or "records" (workgroups' records)."""
    bound, segments = max_context_len or w.max_blocks_per_seq * w.block_size, w.num_seqs * w.num_kv_heads
    if not leaves_records(segments, (bound + BLOCK - 1) // BLOCK, w.head_dim, fp8):
        return "whole"
    return "records" if leaves_records(segments, blocks_of(w).max(), w.head_dim, fp8) else "whole on the device"


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
