"""Offload arrangement of Double Sparsity (Sec. 5.1): the label cache lives on the
GPU, the full K/V caches in pinned host memory, and only the k selected rows of
a layer cross the host link, into one half of a double buffer, while the
previous layer's rows are being attended.

This module only sequences the library's calls on two streams; every step runs
in the library's kernels:
    main stream : ds_select(l + 1)       -> idx[(l + 1) % 2]
                  ds_attend_rows(l)      -> out[l]
    copy stream : ds_gather_rows_host(l) -> rows[l % 2]   (reads pinned host memory)
Row fetch of layer l+1 overlaps the attention of layer l, selection of layer
l+1 the row fetch of layer l.  The paper obtains
layer l+1's query early by pushing layer l's embedding through W_q of layer l+1
(Sec. 5.1); with `predict` the selection does exactly that
(ds_predict_query) and selects with the approximate query, while the attention
uses the layer's real query.  Without it the given queries select, which
exercises the same transport.

The host link is what the step waits for, so only the fetches need a stream of
their own: a layer's selection is enqueued ahead of the previous layer's
attention, which waits for rows anyway.  (With a third stream for the
selection, two of the three could land on one hardware queue and a selection
then waited for a whole fetch; and each layer cost six event calls instead of
four.)
"""
from __future__ import annotations

import torch

from . import binding as ds


class OffloadDecoder:
    def __init__(self, shp: ds.DsShape, device="cuda"):
        self.shp = shp
        self.dev = torch.device(device)
        B, Hq, Hkv, d, k = shp.B, shp.Hq, shp.Hkv, shp.d, shp.k
        self.idx = [torch.empty((B, Hkv, k), dtype=torch.int32, device=self.dev) for _ in range(2)]
        self.rows = [torch.empty((B, Hkv, k, 2, d), dtype=torch.float16, device=self.dev) for _ in range(2)]
        # one workspace for the selections, one for the attention
        self.ws_sel = ds.ds_workspace_alloc(shp, self.dev)
        self.ws_att = ds.ds_workspace_alloc(shp, self.dev)
        self.s_copy = torch.cuda.Stream(device=self.dev)
        self.ev_sel = [torch.cuda.Event() for _ in range(2)]
        self.ev_rows = [torch.cuda.Event() for _ in range(2)]

    def decode(self, layers, outs, predict=None):
        """layers: list of (q, label, channels, K_pinned, V_pinned); outs: list of
        [B,Hq,d] fp32 device tensors.  predict: None, or per layer (x, Wq, q_pred) with
        x [B,Dm] the embedding the prediction starts from, Wq [Hq*d, Dm] the layer's
        query projection and q_pred [B,Hq,d] fp16 receiving the approximate query that
        then selects the layer's rows.  Enqueues one decode step over all layers on the
        current stream (plus the copy stream) and returns without synchronising."""
        main = torch.cuda.current_stream(self.dev)
        n = len(layers)

        # idx[s] and rows[s] are free for layer l when the attention of layer l - 2 is done: the main
        # stream has it ahead of the selection, and the fetch waits for the selection.
        def fetch(l):
            q, label, ch, Kp, Vp = layers[l]
            s = l % 2
            if predict is not None:
                x, Wq, q_pred = predict[l]
                ds.ds_predict_query(x, Wq, q_pred, stream=main)
                q = q_pred
            ds.ds_select(q, label, ch, self.idx[s], self.ws_sel, self.shp, stream=main)
            self.ev_sel[s].record(main)
            self.s_copy.wait_event(self.ev_sel[s])
            ds.ds_gather_rows_host(Kp, Vp, self.idx[s], self.rows[s], self.shp, stream=self.s_copy)
            self.ev_rows[s].record(self.s_copy)

        fetch(0)
        for l in range(n):
            if l + 1 < n:
                fetch(l + 1)
            s = l % 2
            main.wait_event(self.ev_rows[s])
            ds.ds_attend_rows(layers[l][0], self.rows[s], outs[l], self.ws_att, self.shp, stream=main)
