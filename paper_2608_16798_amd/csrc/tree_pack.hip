// Prefix-tree packing of a rollout's model calls (ClawGym II, Sec. 3.2.1; the trainable-token
// rule of Sec. 3.2.3).  Host code only: it turns the captured (context, response) token lists of
// each rollout into the packed positions, parent pointers and training rows that the GPU entry
// points consume.
//
// Tree per rollout: node 0 is the empty root; node 1 holds the first call's context (the task
// prompt, harness content).  A call attaches to the node whose accumulated history is the
// longest prefix of its context, found by a depth-first walk that only follows children whose
// content matches the context at the current offset (a node's history is a prefix of the
// context exactly when every node on its path matches).  The new node holds the context's
// remainder (not trainable) followed by the response (trainable) unless an identical sibling
// exists.  Packing is depth-first pre-order with an explicit stack.
#include <string.h>

#include <new>
#include <vector>

#include "rlk_internal.h"

namespace rlk {
namespace {

// A node's content is a span of the caller's arrays: the context's remainder from its offset on (not
// trainable), then the response (trainable).  Nothing is copied before the packed output is written, which
// takes one pass of copies per node.
struct Node {
  int64_t hist_len = 0;
  const int32_t* x = nullptr;
  int64_t nx = 0;
  const int32_t* y = nullptr;
  int64_t ny = 0;
  std::vector<int> children;
  int64_t size() const { return nx + ny; }
};

bool same_tokens(const int32_t* a, const int32_t* b, int64_t n) {
  return n == 0 || a == b || memcmp(a, b, (size_t)n * sizeof(int32_t)) == 0;
}

// The deepest node whose history is a prefix of x[0, nx); ties go to the earliest node.
int attach_point(const std::vector<Node>& nodes, const int32_t* x, int64_t nx, std::vector<int>& stack) {
  int best = 0;
  int64_t best_len = 0;
  stack.assign(1, 0);
  while (!stack.empty()) {
    const int k = stack.back();
    stack.pop_back();
    const Node& n = nodes[k];
    if (n.hist_len > best_len || (n.hist_len == best_len && k < best)) {
      best = k;
      best_len = n.hist_len;
    }
    for (int c : n.children) {
      const Node& ch = nodes[c];
      const int32_t* at = x + n.hist_len;
      if (n.hist_len + ch.size() <= nx && same_tokens(ch.x, at, ch.nx) && same_tokens(ch.y, at + ch.nx, ch.ny))
        stack.push_back(c);
    }
  }
  return best;
}

void build_tree(const rlk_calls_t* c, int r, std::vector<Node>& nodes, std::vector<int>& stack) {
  nodes.assign(1, Node());
  const int64_t c0 = c->call_off[r], c1 = c->call_off[r + 1];
  if (c1 > c0) {
    const int64_t nx = c->x_off[c0 + 1] - c->x_off[c0];
    if (nx > 0) {
      Node p;
      p.hist_len = nx;
      p.x = c->x_tok + c->x_off[c0];
      p.nx = nx;
      nodes.push_back(std::move(p));
      nodes[0].children.push_back(1);
    }
  }
  for (int64_t k = c0; k < c1; ++k) {
    const int32_t* x = c->x_tok + c->x_off[k];
    const int64_t nx = c->x_off[k + 1] - c->x_off[k];
    const int at = attach_point(nodes, x, nx, stack);
    Node n;
    n.x = x + nodes[at].hist_len;
    n.nx = nx - nodes[at].hist_len;
    n.y = c->y_tok + c->y_off[k];
    n.ny = c->y_off[k + 1] - c->y_off[k];
    n.hist_len = nx + n.ny;
    if (n.size() == 0) continue;
    bool same = false;
    for (int ch : nodes[at].children) {
      const Node& o = nodes[ch];
      if (o.nx == n.nx && o.ny == n.ny && same_tokens(o.x, n.x, n.nx) && same_tokens(o.y, n.y, n.ny)) {
        same = true;
        break;
      }
    }
    if (same) continue;
    nodes.push_back(std::move(n));
    nodes[at].children.push_back((int)nodes.size() - 1);
  }
}

struct Item {
  int node;
  int64_t last;   // packed position of the parent's last token, -1 under the root
  int32_t depth;
};

// Sizes of one rollout's tree: a row per position but the first of each child of the root
void count_tree(const std::vector<Node>& nodes, int64_t& npos, int64_t& nrows) {
  for (const Node& n : nodes) {
    npos += n.size();
    nrows += n.size();
  }
  for (int c : nodes[0].children) nrows -= nodes[c].size() > 0;
}

// Positions and rows of one rollout's tree, appended to the output.
void pack_tree(const std::vector<Node>& nodes, const rlk_tree_out_t* o, int64_t& npos, int64_t& nrows,
               std::vector<Item>& stack) {
  stack.assign(1, {0, -1, 0});
  while (!stack.empty()) {
    const Item it = stack.back();
    stack.pop_back();
    const Node& n = nodes[it.node];
    const int64_t p0 = npos, len = n.size();
    if (len > 0) {
      int32_t* tok = o->token + p0;
      if (n.nx) memcpy(tok, n.x, (size_t)n.nx * sizeof(int32_t));
      if (n.ny) memcpy(tok + n.nx, n.y, (size_t)n.ny * sizeof(int32_t));
      // the first token's parent is the parent node's last token, the others' the token before them
      int32_t* par = o->parent + p0;
      int32_t* dep = o->depth + p0;
      par[0] = (int32_t)it.last;
      for (int64_t i = 1; i < len; ++i) par[i] = (int32_t)(p0 + i - 1);
      for (int64_t i = 0; i < len; ++i) dep[i] = it.depth + (int32_t)i;
      const int64_t skip = it.last < 0 ? 1 : 0;  // no row predicts a tree's first token
      const int64_t q = nrows, m = len - skip, untrained = n.nx > skip ? n.nx - skip : 0;
      if (m > 0) {
        memcpy(o->row_src + q, par + skip, (size_t)m * sizeof(int32_t));
        memcpy(o->row_target + q, tok + skip, (size_t)m * sizeof(int32_t));
        memset(o->row_mask + q, 0, (size_t)untrained);
        memset(o->row_mask + q + untrained, 1, (size_t)(m - untrained));
      }
      npos += len;
      nrows += m;
    }
    // children in first-seen order: push in reverse
    const int64_t last = len > 0 ? npos - 1 : it.last;
    for (size_t i = n.children.size(); i-- > 0;) stack.push_back({n.children[i], last, it.depth + (int32_t)len});
  }
}

}  // namespace
}  // namespace rlk

using namespace rlk;

extern "C" rlk_status_t rlk_tree_pack(const rlk_calls_t* calls, rlk_tree_out_t* out) {
  if (!calls || !out) return report_error(RLK_EINVAL, "calls or out is NULL");
  const int R = calls->R;
  if (R < 0) return report_error(RLK_ESHAPE, "R < 0");
  if (R > 0 && !calls->call_off) return report_error(RLK_EINVAL, "call_off is NULL");
  const int64_t C = R > 0 ? calls->call_off[R] : 0;
  if (R > 0 && calls->call_off[0] != 0) return report_error(RLK_EINVAL, "call_off[0] must be 0");
  for (int r = 0; r < R; ++r)
    if (calls->call_off[r + 1] < calls->call_off[r]) return report_error(RLK_EINVAL, "call_off decreases");
  if (C > 0 && (!calls->x_off || !calls->y_off)) return report_error(RLK_EINVAL, "x_off or y_off is NULL");
  for (int64_t k = 0; k < C; ++k)
    if (calls->x_off[k + 1] < calls->x_off[k] || calls->y_off[k + 1] < calls->y_off[k])
      return report_error(RLK_EINVAL, "x_off or y_off decreases");
  if (C > 0 && ((calls->x_off[C] > calls->x_off[0] && !calls->x_tok) || (calls->y_off[C] > calls->y_off[0] && !calls->y_tok)))
    return report_error(RLK_EINVAL, "token arrays are NULL");
  const bool query = !out->token && !out->parent && !out->depth && !out->pos_off && !out->row_src &&
                     !out->row_target && !out->row_mask && !out->row_cu && !out->leaves;
  if (!query && (!out->token || !out->parent || !out->depth || !out->pos_off || !out->row_src || !out->row_target ||
                 !out->row_mask || !out->row_cu))
    return report_error(RLK_EINVAL, "some output arrays are NULL (all NULL = size query)");
  try {
    // pass 1: sizes
    std::vector<std::vector<Node>> trees(query ? 1 : (size_t)R);
    std::vector<int> walk;
    int64_t npos = 0, nrows = 0;
    for (int r = 0; r < R; ++r) {
      std::vector<Node>& nodes = trees[query ? 0 : r];
      build_tree(calls, r, nodes, walk);
      count_tree(nodes, npos, nrows);
    }
    out->n_pos = npos;
    out->n_rows = nrows;
    if (query) return RLK_OK;
    if (npos > out->cap_pos || nrows > out->cap_rows) return report_error(RLK_ESHAPE, "output capacity too small");
    if (npos > INT32_MAX || nrows > INT32_MAX) return report_error(RLK_ESHAPE, "more than 2^31 packed positions");
    // pass 2: fill
    std::vector<Item> stack;
    npos = nrows = 0;
    out->pos_off[0] = 0;
    out->row_cu[0] = 0;
    for (int r = 0; r < R; ++r) {
      const std::vector<Node>& nodes = trees[r];
      pack_tree(nodes, out, npos, nrows, stack);
      out->pos_off[r + 1] = npos;
      out->row_cu[r + 1] = (int32_t)nrows;
      if (out->leaves) {
        int leaves = 0;
        for (size_t k = 1; k < nodes.size(); ++k) leaves += nodes[k].children.empty();
        out->leaves[r] = leaves;
      }
    }
  } catch (const std::bad_alloc&) {
    return report_error(RLK_ESHAPE, "out of host memory");
  }
  return RLK_OK;
}
