"""Inputs in which some GPUs' decode batch is `batch`: from 31 on every batch reads the last table row,
so a batch of 31 and the largest int32 must give the same results."""
import numpy as np

from paper_2606_30391_amd import workloads as W

INT32_MAX = 2**31 - 1


def placement(batch, R=60, G=40, M=3, NS=8, NF=16, Wn=2, seed=1):
    inp = W.make_tiny_placement(np.random.default_rng(seed), R=R, G=G, M=M, NS=NS, NF=NF, W=Wn, caps=False)
    inp["gpus"]["batch"][:, ::2] = batch
    return inp


def fleet(batch):
    inp = W.make_tiny_fleet(np.random.default_rng(2), G=30, M=3, NS=3, NF=5, loose=True)
    inp["fleet"]["inst_batch"][::2] = batch
    return inp


def llms(batch):
    inp = W.make_tiny_llms(np.random.default_rng(3), G=20, K=3, M=2, NS=4, NF=8)
    inp["llms"]["batch"][::2] = batch
    return inp


def dispatch(batch, S=3):
    inp = W.make_tiny_dispatch(np.random.default_rng(4), R=200, G=12, M=2, NS=3, NF=4, S=S)
    inp["avail"]["batch"][::2] = batch
    return inp


def transfer(batch):
    inp = W.make_transfer(n_gpus=16, requests_per_gpu=6)
    inp["plan"]["batch"][::2] = batch
    return inp
