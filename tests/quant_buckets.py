"""The bucket formula of the quantiser's sort (any4_quantize.hip, sort_by_buckets) on the host, and the limits that the
source states: which rows are sorted into buckets and which go to the bitonic network."""
import os
import re

import numpy as np

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_04610_amd", "csrc",
                      "any4_quantize.hip")


def constants():
    with open(SOURCE) as f:
        text = f.read()
    return {k: int(v) for k, v in re.findall(r"constexpr (?:uint32_t|int) (kBucket\w+) = (\d+);", text)}


def threads(K):
    """of the block that sorts a row of K weights, 16 a thread"""
    return next(t for t in (64, 128, 256, 512, 1024) if K <= 16 * t)


def count(K):
    return 32 * threads(K)


def sizes(ws):
    """elements in every bucket of one scaled row, in the kernel's fp32 arithmetic"""
    ws = np.asarray(ws, np.float32)
    nb = np.float32(count(len(ws)))
    low = ws.min()
    inv = nb / (ws.max() - low)
    at = np.clip((ws - low) * inv, np.float32(0.0), nb - np.float32(1.0)).astype(np.int64)
    return np.bincount(at, minlength=int(nb))


def accepted(ws):
    c = constants()
    n = sizes(ws)
    crowded = n[n > c.get("kBucketOwn", c["kBucketMost"])].astype(np.int64)
    return bool(n.max() <= c["kBucketMost"] and np.sum(crowded * crowded) <= c.get("kBucketLooks", 0) * len(ws))
