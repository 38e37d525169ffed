// The trie's position tables, derived from the string blob and one record per
// string (Section 4.1: one node per distinct prefix; the strings lie in the
// blob in trie order, each after a pad byte that stands for its set's root).
//
//   node_at[p]   the node whose edge byte is blob byte p (a pad: its set's root)
//   depth[g]     the prefix length of node g
//   node_pos[g]  the first blob position of non-root node g: where the string
//                that created it wrote its edge byte (-1 at roots)
//   walk[g]      the node's edge byte (a root: a byte other than T), its other
//                children none yet (see Walk)
//   parent(g)    node_at[node_pos[g] - 1]
//   and under tail compression row_of, tail_span (by node) and row_at (by
//   position), see TailRec
//
// The layout kernel calls the function below with a wave's lanes, and the host
// runs the same function over the host records so that the layout can be
// checked without a GPU.  Every write and every record read is range-checked: an
// inconsistent record, which the host build never makes, is counted instead of
// being followed, and the caller reports the count.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_tables.hpp"

namespace tam {

// Where a layout pass writes (null, from walk on: not kept).
struct LayTables {
    int32_t *node_at, *depth, *node_pos;
    Walk *walk;
    const uint8_t *blob;  // with walk: the strings' bytes
    uint32_t terminator;
    int32_t *row_of, *tail_span, *row_at;
};

// The tables of string record u (one of the records [s0, s1) of a group of whole
// sets), by lane `lane` of `lanes` that share the work.  String u creates the
// nodes first .. first + len - lcp along path indices lcp .. len (depth = index
// + 1); below index lcp its path is an earlier string's: index i belongs to the
// nearest earlier string v of the part with lcp[v] <= i.  Walking from u - 1
// along psv (each step lowers the common prefix), a string whose lcp lies below
// the indices still open owns [lcp[v], open bound); one whose lcp does not is
// passed over.  The chain ends at a string with lcp 0, which owns all that is
// open.  Returns the number of inconsistent record fields met (0 for the host
// build's records).
//   trec: the tail records (null: no tail compression).
//   *parent: the node string u branches off (the one at path index lcp - 1),
//   or -1 for its set's first string, which starts the root's own path.
__host__ __device__ inline int32_t lay_string(const StrRec *strs, const TailRec *trec, int64_t s0, int64_t u,
                                              int64_t blob_bytes, int64_t N, const LayTables &o, int32_t lane,
                                              int32_t lanes, int32_t *parent) {
    const StrRec r = strs[u];
    *parent = -1;
    if (r.at < 0 || r.len < 0 || r.lcp < 0 || r.lcp > r.len || (int64_t)r.at + 1 + r.len >= blob_bytes ||
        r.root < 0 || (int64_t)r.root >= N || r.first <= r.root || (int64_t)r.first + (r.len - r.lcp) >= N)
        return 1;
    const TailRec tr = trec ? trec[u] : TailRec{0, 0, 0, 0};
    const bool opens = r.first == r.root + 1;  // the set's first string
    if (lane == 0) {
        o.node_at[r.at] = r.root;  // the pad stands for the root
        if (o.row_at) o.row_at[r.at] = tr.root;
        if (opens) {
            o.depth[r.root] = 0;
            o.node_pos[r.root] = -1;
            if (o.walk) o.walk[r.root] = Walk{0, o.terminator ^ 1u};
            if (o.row_of) {
                o.row_of[r.root] = tr.root;
                o.tail_span[r.root] = 0;
            }
        }
    }
    for (int32_t i = r.lcp + lane; i <= r.len; i += lanes) {
        const int32_t g = r.first + (i - r.lcp), p = r.at + 1 + i;
        o.node_at[p] = g;
        o.depth[g] = i + 1;
        o.node_pos[g] = p;
        if (o.walk) o.walk[g] = Walk{0, o.blob[p]};
        if (o.row_of) {
            const bool branching = i < tr.next;
            const int32_t row = branching ? tr.row + (i - r.lcp) : -1 - (r.len - i);
            o.row_of[g] = row;
            o.row_at[p] = row;
            o.tail_span[g] = branching ? 0 : i - tr.top;
        }
    }
    if (r.lcp == 0 && !opens) *parent = r.root;
    int32_t hi = r.lcp;  // path indices [0, hi) still open
    int64_t v = u - 1;   // lcp > 0: not the first string of its part
    while (hi > 0) {
        if (v < s0 || v >= u) return 1;  // the chain left the group, or does not go back
        const StrRec q = strs[v];
        if (q.lcp < hi) {
            if (q.lcp < 0 || q.first < 0 || (int64_t)q.first + (hi - 1 - q.lcp) >= N) return 1;
            const TailRec tq = trec ? trec[v] : TailRec{0, 0, 0, 0};
            for (int32_t i = q.lcp + lane; i < hi; i += lanes) {
                const int32_t p = r.at + 1 + i;
                o.node_at[p] = q.first + (i - q.lcp);
                if (o.row_at) o.row_at[p] = i < tq.next ? tq.row + (i - q.lcp) : -1 - (q.len - i);
            }
            if (hi == r.lcp) *parent = q.first + (hi - 1 - q.lcp);
            hi = q.lcp;
        }
        if (q.psv >= v) return 1;  // each step must go back
        v = q.psv;
    }
    return 0;
}

// The parent of non-root node g, or -1 with *bad set when g has no position
// inside the blob or the byte before it is not a node.
__host__ __device__ inline int32_t lay_parent(const int32_t *node_pos, const int32_t *node_at, int64_t N,
                                              int64_t blob_bytes, int64_t g, bool *bad) {
    const int64_t pos = node_pos[g];
    if (pos <= 0 || pos >= blob_bytes) {
        *bad = true;
        return -1;
    }
    const int32_t par = node_at[pos - 1];
    if (par < 0 || (int64_t)par >= N) {
        *bad = true;
        return -1;
    }
    return par;
}

}  // namespace tam
