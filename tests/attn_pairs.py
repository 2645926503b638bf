"""Which form of the decode attention a call takes, from the header that the launch code includes, compiled for the host."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def build(folder):
    exe = os.path.join(str(folder), "attn_pairs_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", os.path.join(HERE, "host", "attn_pairs_check.cpp"), "-o", exe])

    def one_workgroup_per_pair(calls):
        """Per call ("c", pairs, L0, L1, head_dim) or ("p", requests, heads, room of a table row, tokens, head_dim)."""
        out = subprocess.check_output([exe] + [str(v) for c in calls for v in c], text=True)
        return [line == "1" for line in out.split()]
    return one_workgroup_per_pair
